"""Nucleus rows whose cut lies among columns that equal the sampled threshold: the sliced kernels take them with the threshold
above these ties, none is left to the general kernel, whose unit of mass they keep.  Against the oracle."""
import math

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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_masses_keep_the_unit_of_the_general_kernel(dtype):
    """Masses of such rows are integers in units of 2^-43 of the largest one, as the general kernel's are: V roundings of half a unit
    and the weights' relative error below 1e-12, whatever the threshold.  (Most columns share one value here, so that their
    roundings add up instead of cancelling.  The threshold is the second level's value, since it aims at more than 1024 columns, and the
    cut lies among that level's.)"""
    B, V, nnz = 32, 131_072, 16
    rng = np.random.default_rng(11)
    z = np.empty((B, V), np.float32)
    for b in range(B):
        z[b, rng.permutation(V)] = np.where(np.arange(V) < 1000, 0.0, np.where(np.arange(V) < 3000, -0.25 - 0.25 * (b % 4), -14.0 - 0.0625 * b))
    hist_ptr = np.arange(B + 1, dtype=np.int64) * nnz
    hist_ids = rng.integers(0, V, B * nnz).astype(np.int32)
    params = synth.make_params(B, temperature=1.0, top_p=np.linspace(0.65, 0.9, B).astype(np.float32), freq_penalty=0.1, n_prompt=nnz // 2)
    bits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    w = synth.Workload("unit", B, V, dtype, bits, params, hist_ptr, hist_ids)
    ids, dg = P.run_gpu(w, 0)
    P.compare(ids, dg, P.run_oracle(w, 0), range(B))
    assert (dg["flags"] & binding.DIAG_WIDE).all()
    for b in range(B):
        y = w.logits_f32()[b].copy()
        gen, count = np.unique(hist_ids[b * nnz + nnz // 2:(b + 1) * nnz], return_counts=True)
        y[gen] -= np.float32(0.1) * count.astype(np.float32)
        s_k = math.fsum(np.exp(y.astype(np.float64) - y.max()))  # (a running sum in float64 is off by more)
        off = float(dg["s_k"][b]) - s_k
        assert abs(off) <= V * 2.0 ** -44 + 1e-12 * s_k, (b, off, s_k)
