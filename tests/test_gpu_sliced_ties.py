"""Nuclei that end among thousands of equal values, wider than the candidate list: the finishing kernel divides the
ids of one value, and the drawn slice is the row's first, a middle or its ragged last one.  Against the oracle."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype,pad", [(32_768, "f32", 0), (40_963, "f32", 1), (32_777, "bf16", 7), (65_535, "bf16", 1)])
@pytest.mark.parametrize("ties", [300, 513, 1100, 3900])
def test_cut_among_ties(V, dtype, pad, ties):
    rng = np.random.default_rng(V + ties)
    B = 12
    z = np.empty((B, V), np.float32)
    for b in range(B):
        order = rng.permutation(V) if b % 3 else np.arange(V)  # every third row: equal values side by side
        z[b, order] = 6.0 - 0.25 * (np.arange(V) // ties).clip(0, 40)
    hist_ptr = np.arange(B + 1, dtype=np.int64) * 200
    hist_ids = rng.integers(0, V, B * 200).astype(np.int32)  # penalties keep bfloat16 rows off the counts per pattern
    params = synth.make_params(B, temperature=rng.choice([0.7, 1.0], B).astype(np.float32), top_p=rng.choice([0.5, 0.9, 0.99], B).astype(np.float32),
                               rep_penalty=1.1, freq_penalty=0.1, pres_penalty=0.1, n_prompt=50)
    bits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    w = synth.Workload("ties", B, V, dtype, bits, params, hist_ptr, hist_ids,
                       hot_ids=np.sort(rng.choice(V, V // 8, replace=False)).astype(np.int32) if pad else None)
    for step in range(2):
        ids, dg = P.run_gpu(w, step)
        assert not (dg["flags"] & binding.DIAG_ERROR).any()
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
