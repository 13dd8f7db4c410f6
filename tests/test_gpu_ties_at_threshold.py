"""Nucleus rows whose cut lies among columns that equal the sampled threshold: the sliced kernels take them with the threshold
above these ties, none is left to the general kernel.  Against the oracle."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,hot,shift", [(60_000, False, 0.0), (60_003, True, -6.0), (131_072, False, -40.0)])
def test_cut_among_ties_at_g(dtype, V, hot, shift):
    B, nnz = 96, 40
    rng = np.random.default_rng(V)
    z = np.full((B, V), -12.0, np.float32)
    for b in range(B):  # steps of about 300 columns each, a quarter apart: any threshold is the value of one step
        step = np.minimum(np.arange(V) // 300, 40).astype(np.float32)
        z[b, rng.permutation(V)] = -0.25 * step - np.where(step >= 40, 6.0, 0.0)
    z += np.float32(shift)
    hist_ptr = np.arange(B + 1, dtype=np.int64) * nnz
    hist_ids = rng.integers(0, V, B * nnz).astype(np.int32)
    # prefixes of 900 to 3000 columns: the masses of the steps are those of a geometric series
    top_p = np.linspace(0.45, 0.9, B).astype(np.float32)
    params = synth.make_params(B, temperature=1.0, top_p=top_p, rep_penalty=1.1, freq_penalty=0.1, pres_penalty=0.1, n_prompt=nnz // 2)
    bits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    w = synth.Workload("ties", B, V, dtype, bits, params, hist_ptr, hist_ids,
                       hot_ids=np.sort(rng.choice(V, V // 8, replace=False)).astype(np.int32) if hot else None)
    for step in range(2):
        ids, dg = P.run_gpu(w, step)
        assert not (dg["flags"] & (binding.DIAG_ERROR | binding.DIAG_GENERAL)).any()
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
