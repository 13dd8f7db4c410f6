"""Rows with a nucleus wider than the candidate list: float32 rows and calls of few rows slice by slice (test_runs), and calls
whose workgroups take enough of a bfloat16 row's slices in runs of them (test_rows_in_runs): history columns settled behind the run,
columns by their patterns, groups with values that have no entry column by column.  Against the oracle."""
import os
import re

import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


def rows_of(rng, B, V, hist_ids, nnz, dtype):
    """Six kinds of rows: ordinary; zeros and tiny values; magnitudes beyond 256; masked columns of three sorts; history
    columns far above the others as read, far below as penalised; values of one binade, so that many tie."""
    z = np.empty((B, V), np.float32)
    tau = np.ones(B, np.float32)
    pres = np.full(B, 0.2, np.float32)
    for b in range(B):
        z[b, rng.permutation(V)] = -1.1 * np.log1p(np.arange(V))
        z[b] += rng.normal(0.0, 1.5, V)
        kind = b % 6
        if kind == 1:
            z[b] += 6.0
            z[b, rng.random(V) < 0.2] = 0.0
            tiny = rng.random(V) < 0.01
            z[b, tiny] = rng.choice([1e-6, -3e-5, 1e-30, -0.0], int(tiny.sum()))
        elif kind == 2:
            z[b] *= 40.0
            tau[b] = 40.0
        elif kind == 3:
            u = rng.random(V)
            z[b, u < 0.2] = -np.inf
            z[b, (u >= 0.2) & (u < 0.3)] = -1e4
            z[b, (u >= 0.3) & (u < 0.31)] = -3.38e38
        elif kind == 4:
            z[b, hist_ids[b * nnz:(b + 1) * nnz]] += 30.0
            pres[b] = 60.0
        elif kind == 5:
            z[b] = 96.0 + z[b].clip(-30.0, 30.0)
    return z, tau, pres


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,B,nnz,hot", [(32_771, 18, 300, False), (40_960, 24, 20_000, True), (150_001, 48, 2500, True),
                                         (150_007, 48, 2500, False), (9_221, 12, 1, False)])
def test_runs(dtype, V, B, nnz, hot):
    if dtype == "bf16" and V < 16_384:
        V += 16_384  # (shorter bfloat16 rows are the general kernel's)
    rng = np.random.default_rng(V + nnz)
    hist_ptr = np.arange(B + 1, dtype=np.int64) * nnz
    hist_ids = rng.integers(0, V, B * nnz).astype(np.int32)
    hist_ids[::max(nnz // 2, 1)] = V - 1  # the last column, behind the last whole group
    z, tau, pres = rows_of(rng, B, V, hist_ids, nnz, dtype)
    top_p = rng.choice([0.8, 0.95, 0.99], B).astype(np.float32)
    params = synth.make_params(B, temperature=tau, top_p=top_p, min_p=np.where(np.arange(B) % 4 == 3, 1e-4, 0.0).astype(np.float32),
                               rep_penalty=1.1, freq_penalty=0.1, pres_penalty=pres, n_prompt=nnz // 3)
    bits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    w = synth.Workload("runs", B, V, dtype, bits, params, hist_ptr, hist_ids,
                       hot_ids=np.sort(rng.choice(V, V // 8, replace=False)).astype(np.int32) if hot else None)
    wide = 0
    for step in range(2):
        ids, dg = P.run_gpu(w, step)
        assert not (dg["flags"] & binding.DIAG_ERROR).any()
        wide += int(((dg["flags"] & binding.DIAG_WIDE) != 0).sum())
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
    assert wide > B // 2


def run_rule():
    """The constants of takes_run: with h history columns a slice, at most RUN_MAX_IDS, a row is taken in runs from RUN_MIN + h / RUN_IDS
    slices a workgroup, but for pieces of fewer than RUN_PIECE slices."""
    src = open(os.path.join(os.path.dirname(binding.__file__), "csrc", "simple_wide.hip")).read()
    return [int(x) for x in re.search(r"RUN_MIN = (\d+), RUN_IDS = (\d+), RUN_MAX_IDS = (\d+), RUN_PIECE = (\d+)", src).groups()]


@pytest.mark.parametrize("V,chunk,nnz,hot", [(17_003, 16, 60, True), (28_675, 13, 300, True), (40_960, 15, 700, False), (150_001, 21, 2500, True), (150_008, 30, 2500, False)])
def test_rows_in_runs(V, chunk, nnz, hot):
    """Nine rows, repeated until a workgroup takes `chunk` slices: pieces of a row long enough for a run, and shorter ones.  The first
    nine and the last go through the oracle; masses are integers, so every copy of a row has the first one's, however it was cut."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    SLC, K = 4096, 9
    n_sl = -(-V // SLC)
    B = -(-chunk * 4 * n_cu // (n_sl * K)) * K
    rng = np.random.default_rng(V + nnz)
    ids9 = rng.integers(0, V, K * nnz).astype(np.int32)
    ids9[::max(nnz // 2, 1)] = V - 1  # the last column, behind the last whole group
    z9, tau9, pres9 = rows_of(rng, K, V, ids9, nnz, "bf16")
    z9[6] += 300.0   # no value has an entry
    z9[7] -= 300.0
    z9[8] = z9[8] / 4.0 + 232.0  # (of kind 2) the largest have none
    tau9[8] = 10.0
    params9 = synth.make_params(K, temperature=tau9, top_p=rng.choice([0.8, 0.95, 0.99], K).astype(np.float32),
                                min_p=np.where(np.arange(K) == 3, 1e-4, 0.0).astype(np.float32), rep_penalty=1.1, freq_penalty=0.1,
                                pres_penalty=pres9, n_prompt=nnz // 3)
    times = B // K
    tile = lambda x: np.tile(x, (times,) + (1,) * (x.ndim - 1))
    hot_ids = np.sort(rng.choice(V, V // 8, replace=False)).astype(np.int32) if hot else None
    w = synth.Workload("in runs", B, V, "bf16", tile(synth.f32_to_bf16_bits(z9)), tile(params9), np.arange(B + 1, dtype=np.int64) * nnz, tile(ids9), hot_ids=hot_ids)
    dev = P.to_device(w)
    padded = torch.zeros(B, -(-V // 8) * 8, dtype=torch.bfloat16, device="cuda:0")  # (rows at 16-byte boundaries)
    padded[:, :V] = dev["logits"]
    dev["logits"] = padded[:, :V]
    ids, dg = P.run_gpu(w, 1, dev=dev)
    assert not (dg["flags"] & binding.DIAG_ERROR).any()
    ends = list(range(K)) + list(range(B - K, B))
    P.compare(ids, dg, P.run_oracle(w, 1, rows=ends), ends)
    for f in ("s_k", "n_survivors", "alpha"):
        assert np.array_equal(dg[f].reshape(times, K), np.broadcast_to(dg[f][:K], (times, K)), equal_nan=f == "alpha"), f
    # slices a workgroup took, and what runs need
    wide = int(((dg["flags"] & binding.DIAG_WIDE) != 0).sum())
    run_min, run_ids, run_max_ids, run_piece = run_rule()
    per_slice = max(len(np.unique(ids9[b * nnz:(b + 1) * nnz])) for b in range(K)) // n_sl
    assert per_slice <= run_max_ids and min(chunk, n_sl) >= run_piece and -(-wide * n_sl // (4 * n_cu)) >= run_min + per_slice // run_ids, (wide, B)
    assert wide >= B // 2
