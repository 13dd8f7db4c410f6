"""Temperature sampling without truncation against the oracle: any dynamic range (one column may hold
almost all of the mass), masked columns, penalties, hot sets, ragged slices, few and many rows."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V,B", [("f32", 8192, 5), ("f32", 12_289, 40), ("f32", 40_963, 300), ("f32", 128_256, 20),
                                       ("bf16", 16_385, 40), ("bf16", 40_968, 300), ("f32", 270_001, 8), ("bf16", 524_287, 4)])
@pytest.mark.parametrize("history,hot_set", [(False, False), (False, True), (True, False), (True, True)])
def test_every_column_survives(dtype, V, B, history, hot_set):
    rng = np.random.default_rng(V + 2 * history + hot_set)
    n_kinds = 8
    z = synth.zipf_profile_logits(n_kinds, V, 1.1, 1.5, rng, "f32", rng.permutation(V))
    z[1, V // 2] = z[1].max() + 40.0                                      # one column holds almost everything
    z[2, rng.choice(V, 3, replace=False)] = z[2].max() + np.float32(17.0)  # three do
    z[3, rng.permutation(V)[:V - 50]] = -np.inf                           # fifty columns left
    z[4, : V // 2] = -np.inf
    z[5] = rng.standard_normal(V) * 0.01                                  # almost uniform
    z[6] = rng.standard_normal(V) * 40.0                                  # range far beyond float32 exponentials
    z[7, V - 1] = z[7].max() + 5.0                                        # the last column, in a ragged group
    kind = np.arange(B) % n_kinds
    z = z[kind]
    logits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    lens = rng.integers(1, 2000, B) if history else np.zeros(B, np.int64)
    hist_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    hist_ids = np.concatenate([np.where(rng.random(int(n)) < 0.5, rng.integers(0, V, int(n)), rng.integers(0, min(V, 3000), int(n)))
                               for n in lens]).astype(np.int32)           # some slices hold most of a history
    pen = dict(rep_penalty=1.1, freq_penalty=0.2, pres_penalty=0.1, n_prompt=50) if history else {}
    params = synth.make_params(B, temperature=rng.choice(np.array([0.5, 0.7, 1.0, 1.4], np.float32), B), **pen)
    hot = np.sort(rng.choice(V, V // 5, replace=False)).astype(np.int32) if hot_set else None
    w = synth.Workload(f"all-{dtype}-{V}", B, V, dtype, logits, params, hist_ptr, hist_ids, hot_ids=hot)
    rows = list(range(B)) if B <= 40 else sorted(rng.choice(B, 32, replace=False).tolist())
    for step in (0, 1):
        ids, dg = P.run_gpu(w, step)
        P.compare(ids, dg, P.run_oracle(w, step, rows=rows), rows)
        assert not (dg["flags"] & (binding.DIAG_ERROR | binding.DIAG_GENERAL)).any()
        assert (dg["n_survivors"] == V).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_that_cannot_be_sampled_are_reported(dtype):
    V, B = 20_000, 6
    rng = np.random.default_rng(5)
    z = rng.standard_normal((B, V)).astype(np.float32)
    z[1, 777] = np.nan
    z[2, 19_999] = np.inf
    z[3] = -np.inf
    z[4, :] = np.float32(1e30)  # finite, but the tempered value overflows at a temperature of 1e-9
    params = synth.make_params(B, temperature=np.array([1, 1, 1, 1, 1e-9, 1], np.float32))
    logits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    w = synth.Workload("all-errors", B, V, dtype, logits, params, np.zeros(B + 1, np.int64), np.zeros(0, np.int32))
    ids, dg = P.run_gpu(w, 0)
    err = (dg["flags"] & binding.DIAG_ERROR) > 0
    assert err.tolist() == [False, True, True, True, True, False] and (ids[err] == -1).all()
    P.compare(ids, dg, P.run_oracle(w, 0, rows=[0, 5]), [0, 5])
