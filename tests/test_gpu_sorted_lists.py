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
