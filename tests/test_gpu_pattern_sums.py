"""The pattern-count kernel's sums at their limits, against the oracle: every column of a lane at the largest mass, every
column of a lane in a cut pattern of which a part survives (the largest count a sum of four takes), patterns at
the ends of the table on either side of zero, rows that end on a tile, one column behind it and one before it."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

# (a dyadic share of equal masses: the cut is exact in float64 sums and in the kernel's integers)
CONTROLS = [dict(top_p=0.5), dict(top_p=0.875), dict(), dict(min_p=0.5), dict(top_p=0.5, temperature=0.5), dict(top_p=0.03125)]
SMALLEST = 2.0 ** -14 * 1.015625  # the smallest magnitude with a bin of its own; 255 is the largest
# No row's cut falls into the bins that zeros share, and with 12 as the maximum what these cost is below a 2^-28th of the
# mass (e^-12 6.2e-5 = 3.8e-10), so that the kernel completes every one of them.
ENDS = [[12.0, 12.0, SMALLEST, -SMALLEST, 0.0, -0.0, -255.0, -256.0],
        [SMALLEST, -SMALLEST, -255.0, -256.0],  # masses of both inner ends within a cut's reach
        [255.0, 254.0, SMALLEST, -SMALLEST, 0.0, -255.0]]


@pytest.mark.parametrize("hot", [False, True])
@pytest.mark.parametrize("V", [24_576, 24_577, 26_623])  # 12 tiles, and a column more; 13 and a column less
@pytest.mark.parametrize("values", ["equal", "signs", "ends"])
def test_sums_at_their_limits(values, V, hot):
    rng = np.random.default_rng(V + len(values))
    B = len(CONTROLS)
    z = np.empty((B, V), np.float32)
    for b in range(B):
        z[b] = {"equal": np.full(V, 3.0 if b % 2 else -3.0), "signs": rng.choice([1.5, -1.5], V),
                "ends": rng.choice(np.array(ENDS[b % len(ENDS)], np.float32), V)}[values]
    base = dict(temperature=1.0, top_p=1.0, min_p=0.0)
    cols = {k: np.array([c.get(k, v) for c in CONTROLS], np.float32) for k, v in base.items()}
    w = synth.Workload("sums", B, V, "bf16", synth.f32_to_bf16_bits(z), synth.make_params(B, **cols), np.zeros(B + 1, np.int64),
                       np.zeros(0, np.int32), hot_ids=np.sort(rng.choice(V, V // 3, replace=False)).astype(np.int32) if hot else None)
    for step in range(2):
        ids, dg = P.run_gpu(w, step)
        assert not (dg["flags"] & binding.DIAG_ERROR).any()
        assert ((dg["flags"] & binding.DIAG_PATTERN) > 0).all()
        P.compare(ids, dg, P.run_oracle(w, step), range(B))
