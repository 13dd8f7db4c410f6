"""Candidate lists at the sizes where their epilogue changes its way, against the oracle: ranked by counting
(up to 128 entries) or by buckets (up to 2048), decided by one wave (up to 64 entries that may survive) or by
all, left to the bucket tables (longer, or crowded by ties).  Masked rows give lists of an exact length."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

CONTROLS = [dict(), dict(top_p=0.9), dict(top_k=64, top_p=0.95), dict(top_k=65), dict(top_k=1), dict(min_p=0.02), dict(top_k=128, min_p=0.001),
            dict(top_k=129, top_p=0.99), dict(top_k=1000, top_p=0.999), dict(temperature=0.0), dict(top_p=0.0), dict(temperature=0.02, top_k=500),
            dict(temperature=0.02, top_p=0.9999, min_p=1e-6), dict(top_k=1024)]


@pytest.mark.parametrize("V,dtype", [(700, "f32"), (4000, "f32"), (4000, "bf16"), (50_000, "f32"), (50_000, "bf16")])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 512, 513, 2047, 2048, 2049])
@pytest.mark.parametrize("values,hot", [("spread", False), ("spread", True), ("ties", False), ("equal", True)])
def test_list_lengths(V, dtype, n, values, hot):
    if n > V:
        pytest.skip("a row has no so many columns")
    B = len(CONTROLS)
    rng = np.random.default_rng(V + 3 * n + len(values))
    z = np.full((B, V), -np.inf, np.float32)
    for b in range(B):
        ids = rng.choice(V, n, replace=False)
        z[b, ids] = {"spread": 2.5 * rng.standard_normal(n), "ties": rng.integers(0, 4, n) * 0.5, "equal": np.ones(n)}[values]
    base = dict(temperature=1.0, top_k=0, top_p=1.0, min_p=0.0)
    cols = {k: np.array([c.get(k, v) for c in CONTROLS], np.int32 if k == "top_k" else np.float32) for k, v in base.items()}
    w = synth.Workload("lists", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, synth.make_params(B, **cols),
                       np.zeros(B + 1, np.int64), np.zeros(0, np.int32),
                       hot_ids=np.sort(rng.choice(V, max(1, V // 5), replace=False)).astype(np.int32) if hot else None)
    for step in range(2):
        ids, dg = P.run_gpu(w, step)
        assert not (dg["flags"] & binding.DIAG_ERROR).any()
        P.compare(ids, dg, P.run_oracle(w, step), range(B))


@pytest.mark.parametrize("V,dtype", [(50_000, "f32"), (151_936, "bf16"), (262_145, "f32"), (500_001, "bf16")])
@pytest.mark.parametrize("n", [256, 257, 300, 511, 512, 513, 1100, 2048])
@pytest.mark.parametrize("hot", [False, True])
def test_neighbouring_ids(V, dtype, n, hot):
    """Survivors side by side: more of them in the draw's range of ids than are resolved at once."""
    B = 12
    rng = np.random.default_rng(V + n)
    z = np.full((B, V), -np.inf, np.float32)
    for b in range(B):
        start = [0, V - n, int(rng.integers(0, V - n)), 1 << 15][b % 4]
        start = min(start, V - n)
        z[b, start:start + n] = rng.standard_normal(n) if b % 3 else rng.integers(0, 900, n) / 256.0
    params = synth.make_params(B, temperature=np.resize(np.array([1.0, 2.0], np.float32), B), top_k=np.resize(np.array([1024, min(n, 1024), 0], np.int32), B),
                               top_p=np.resize(np.array([1.0, 0.999, 0.9999], np.float32), B), min_p=np.resize(np.array([0.0, 0.0, 1e-4, 0.0], np.float32), B))
    w = synth.Workload("neighbours", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params, np.zeros(B + 1, np.int64),
                       np.zeros(0, np.int32), hot_ids=np.sort(rng.choice(V, V // 3, replace=False)).astype(np.int32) if hot else None)
    for step in range(2):
        ids, dg = P.run_gpu(w, step)
        assert not (dg["flags"] & (binding.DIAG_ERROR | binding.DIAG_GENERAL)).any(), params["top_k"][(dg["flags"] & binding.DIAG_GENERAL) > 0]
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
