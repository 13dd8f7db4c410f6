"""Greedy and top-k rows whose large or finite logits lie where a sample of the row misjudges them, against the oracle:
the candidate list still holds them, no row is left to the general kernel.  Few rows (1024 threads each) and more than
the compute units (512 threads)."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

TOP_K = [1, 5, 20, 50, 100, 300]
SHAPES = [(151_936, "bf16"), (128_256, "f32"), (262_144, "bf16")]


def _check(name, make_row, V, dtype, B, history=0, top_k=TOP_K):
    """make_row(rng, b) -> V float32 logits.  Every seventh row is greedy; the oracle decides a sample of the rows."""
    rng = np.random.default_rng(V + B + len(name))
    bits = np.empty((B, V), np.uint16 if dtype == "bf16" else np.float32)
    for b in range(B):
        z = np.asarray(make_row(rng, b), np.float32)
        bits[b] = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    temperature = np.where(np.arange(B) % 7 == 6, 0.0, rng.choice([0.6, 1.0, 1.3], B)).astype(np.float32)
    params = synth.make_params(B, temperature=temperature, top_k=np.resize(np.array(top_k, np.int32), B),
                               top_p=np.resize(np.array([1.0, 0.9, 0.95, 1.0], np.float32), B), rep_penalty=1.1 if history else 1.0,
                               freq_penalty=0.1 if history else 0.0, n_prompt=history // 2)
    w = synth.Workload(name, B, V, dtype, bits, params, np.arange(B + 1, dtype=np.int64) * history, rng.integers(0, V, B * history).astype(np.int32))
    ids, dg = P.run_gpu(w, 0)
    assert not (dg["flags"] & binding.DIAG_ERROR).any()
    rows = sorted(set(range(min(B, 14))) | set(range(0, B, 41)))
    P.compare(ids[rows], dg[rows], P.run_oracle(w, 0, rows=rows), range(len(rows)))
    handed = np.flatnonzero(dg["flags"] & binding.DIAG_GENERAL)
    assert handed.size == 0, f"{handed.size} rows left to the general kernel, top-k {sorted(set(params['top_k'][handed]))}"


def _profile(V):
    return (-1.1 * np.log(np.arange(1, V + 1))).astype(np.float32)


def _noise(rng, n, sigma):
    return rng.standard_normal(n, dtype=np.float32) * np.float32(sigma)


@pytest.mark.parametrize("V,dtype", SHAPES)
@pytest.mark.parametrize("B", [14, 270])
@pytest.mark.parametrize("masked", ["tail 0.07", "tail 0.5", "random 0.5", "random 0.95"])
def test_columns_masked_with_the_lowest_value(V, dtype, B, masked):
    """The lowest finite value (a row in three: another large negative one) among the sample's values."""
    kind, share = masked.split()
    base = _profile(V)
    lowest = synth.bf16_bits_to_f32(np.array([0xFF7F], np.uint16))[0] if dtype == "bf16" else np.finfo(np.float32).min

    def row(rng, b):
        z = base[rng.permutation(V)] + _noise(rng, V, 1.5)
        where = np.arange(V) >= int(V * (1.0 - float(share))) if kind == "tail" else rng.random(V, dtype=np.float32) < float(share)
        return np.where(where, np.float32(-1e30) if b % 3 == 2 else lowest, z)

    _check(masked, row, V, dtype, B, history=200 if kind == "random" else 0)


@pytest.mark.parametrize("V,dtype", SHAPES + [(50_001, "f32")])
@pytest.mark.parametrize("B", [14, 270])
@pytest.mark.parametrize("order", ["frequency", "reversed", "blocks"])
def test_ids_in_order_of_frequency(V, dtype, B, order):
    """As a trained vocabulary has them: the first tile of a row holds most of its large logits."""
    base = _profile(V)

    def row(rng, b):
        if order == "blocks":  # in order of frequency by thousands, any order inside
            return base[np.lexsort((rng.random(V, dtype=np.float32), np.arange(V) // 1000))] + _noise(rng, V, 1.5)
        return (base if order == "frequency" else base[::-1]) + _noise(rng, V, 1.5)

    _check(order, row, V, dtype, B, history=200 if order == "blocks" else 0)


@pytest.mark.parametrize("V,dtype", SHAPES)
@pytest.mark.parametrize("B", [14, 270])
@pytest.mark.parametrize("allowed,runs", [(300, 1), (1000, 1), (3000, 1), (6000, 1), (3200, 100)])
def test_runs_of_allowed_ids(V, dtype, B, allowed, runs):
    """Allow-lists of neighbouring ids, at any place of the row; -inf elsewhere."""
    def row(rng, b):
        z = np.full(V, -np.inf, np.float32)
        n = allowed // runs
        for start in rng.choice(V // n, runs, replace=False) * n if runs > 1 else [rng.integers(0, V - n)]:
            z[start:start + n] = _noise(rng, n, 2.0)
        return z

    _check(f"runs-{allowed}-{runs}", row, V, dtype, B)


@pytest.mark.parametrize("V,dtype", [(128_256, "f32"), (151_936, "bf16")])
@pytest.mark.parametrize("B", [14, 270])
def test_a_raised_band(V, dtype, B):
    """Three thousand neighbouring ids far above the rest, which is finite."""
    def row(rng, b):
        z = _noise(rng, V, 1.0)
        start = int(rng.integers(0, V - 3000))
        z[start:start + 3000] += np.float32(8.0)
        return z

    _check("band", row, V, dtype, B)


def test_most_of_the_largest_in_the_sample():
    """25 of a row's 50 largest columns in the sampled tiles (eight waves' first two; 13 are expected), each in another of
    the 64 groups of eight lanes: the rank asked for lies beyond them."""
    V, tile, waves = 128_256, 2048, 8
    starts = [(w * (V // tile) // waves) * tile for w in range(waves)]
    outside = np.setdiff1d(np.arange(V), np.concatenate([np.arange(s, s + 2 * tile) for s in starts]))

    def row(rng, b):
        z = _noise(rng, V, 1.0)
        group = rng.choice(64, 25, replace=False)
        lane = 8 * (group % 8) + rng.integers(0, 8, 25)
        z[np.array(starts)[group // 8] + rng.integers(0, 2, 25) * tile + rng.integers(0, 4, 25) * 512 + lane * 8 + rng.integers(0, 8, 25)] = 20.0 + rng.random(25)
        z[rng.choice(outside, 24, replace=False)] = 18.0 + rng.random(24)
        return z

    _check("crowded-sample", row, V, "bf16", 270, top_k=[50])
