"""Rows that start at any element's address (odd vocabularies stored without padding, a logits pointer
into the middle of a buffer) against the oracle: every route of the call reads them in 16-byte groups."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V,offset,B", [
    ("f32", 8193, 1, 9), ("f32", 33_001, 3, 9), ("f32", 50_001, 0, 300), ("f32", 65_539, 2, 600),
    ("bf16", 16_385, 1, 9), ("bf16", 40_007, 7, 9), ("bf16", 50_001, 0, 300), ("bf16", 33_002, 5, 600)])
@pytest.mark.parametrize("history", [False, True])
def test_rows_at_any_element(dtype, V, offset, B, history):
    import torch
    rng = np.random.default_rng(V + offset + history)
    z = synth.zipf_profile_logits(B, V, 1.1, 1.5, rng, "f32", rng.permutation(V))
    z[1::9] = rng.standard_normal((z[1::9].shape[0], V)) * 1.2        # nuclei wider than the candidate list
    logits = synth.f32_to_bf16_bits(z) if dtype == "bf16" else z
    controls = dict(temperature=np.resize([1.0, 1.1, 0.0, 0.8, 0.9, 1.0, 1.0, 0.7, 1.2], B).astype(np.float32),
                    top_k=np.resize([0, 0, 0, 50, 0, 1000, 0, 3000, 20], B).astype(np.int32),
                    top_p=np.resize([0.9, 0.95, 1.0, 0.9, 1.0, 0.97, 1.0, 1.0, 1.0], B).astype(np.float32),
                    min_p=np.resize([0, 0, 0, 0, 0.02, 0, 0, 0, 0.05], B).astype(np.float32))
    lens = rng.integers(1, 900, B) if history else np.zeros(B, np.int64)
    if history:
        controls.update(rep_penalty=1.1, freq_penalty=0.2, pres_penalty=0.1, n_prompt=100)
    head = np.argpartition(-z, 2000, axis=1)[:, :2000]
    hist_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    hist_ids = np.concatenate([rng.choice(head[b], int(lens[b])) for b in range(B)]).astype(np.int32)
    hot = np.sort(rng.choice(V, V // 8, replace=False)).astype(np.int32) if offset % 2 else None
    w = synth.Workload(f"unaligned-{dtype}-{V}", B, V, dtype, logits, synth.make_params(B, **controls), hist_ptr, hist_ids, hot_ids=hot)
    # the rows lie back to back in a larger buffer; NaN around them must never be read as a logit
    flat = np.full(B * V + 16, np.nan, np.float32) if dtype == "f32" else np.full(B * V + 16, 0x7FC0, np.uint16)
    flat[offset:offset + B * V] = logits.reshape(-1)
    dev = P.to_device(w)
    buf = torch.from_numpy(flat if dtype == "f32" else flat.view(np.int16)).cuda()
    buf = buf if dtype == "f32" else buf.view(torch.bfloat16)
    dev["logits"] = buf[offset:offset + B * V].view(B, V)
    rows = list(range(B)) if B <= 9 else sorted(rng.choice(B, 27, replace=False).tolist())
    ids, dg = P.run_gpu(w, 3, dev=dev)
    P.compare(ids, dg, P.run_oracle(w, 3, rows=rows), rows)
    assert not (dg["flags"] & binding.DIAG_ERROR).any()
    # the general kernel only completes what the others hand on (one row of nine: top-k 3000 or a sampled threshold that missed)
    assert ((dg["flags"] & binding.DIAG_GENERAL) > 0).mean() <= 0.12


@pytest.mark.parametrize("dtype,V,offset,B", [("f32", 20_001, 1, 8), ("f32", 20_000, 0, 300), ("f32", 17_500, 0, 700), ("bf16", 33_001, 3, 8),
                                              ("bf16", 50_048, 0, 700)])
@pytest.mark.parametrize("gaussian", [False, True])
def test_long_top_k_on_short_rows(dtype, V, offset, B, gaussian):
    """Top-k 600 to 1000 on rows whose sample hands over fewer values than the threshold's rank."""
    import torch
    rng = np.random.default_rng(V + gaussian)
    z = rng.standard_normal((B, V)).astype(np.float32) if gaussian else synth.zipf_profile_logits(B, V, 1.1, 1.5, rng, "f32", rng.permutation(V))
    params = synth.make_params(B, temperature=0.9, top_k=np.resize([1000, 600, 800], B).astype(np.int32), top_p=0.99)
    w = synth.Workload("long-k", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params, np.zeros(B + 1, np.int64), np.zeros(0, np.int32))
    dev = P.to_device(w)
    if offset:
        buf = torch.zeros(B * V + 16, dtype=dev["logits"].dtype, device="cuda:0")
        buf[offset:offset + B * V] = dev["logits"].reshape(-1)
        dev["logits"] = buf[offset:offset + B * V].view(B, V)
    ids, dg = P.run_gpu(w, 0, dev=dev)
    rows = sorted(rng.choice(B, min(B, 24), replace=False).tolist())
    P.compare(ids, dg, P.run_oracle(w, 0, rows=rows), rows)
    print((V, gaussian), "general:", ((dg["flags"] & binding.DIAG_GENERAL) > 0).mean(), flush=True)
    assert ((dg["flags"] & binding.DIAG_GENERAL) > 0).mean() <= 0.05
