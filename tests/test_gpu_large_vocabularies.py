"""Vocabularies around 2^18 columns and up to where only the general kernel serves a call (2^19): every
route of the single-pass, sliced and pattern-count kernels against the oracle."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V,B,hot_share", [
    ("f32", (1 << 18) - 1, 10, 0.0), ("f32", 1 << 18, 300, 0.1), ("f32", 270_001, 600, 0.0), ("f32", (1 << 19) - 1, 10, 0.1),
    ("bf16", 1 << 18, 10, 0.1), ("bf16", 270_001, 300, 0.0), ("bf16", 300_008, 600, 0.1), ("bf16", (1 << 19) - 1, 10, 0.0),
    ("f32", 1 << 19, 4, 0.0), ("bf16", 1 << 19, 4, 0.1)])
def test_routes_on_large_vocabularies(dtype, V, B, hot_share):
    import torch
    rng = np.random.default_rng(V % 977 + B)
    n_kinds = 10  # rows repeat ten profiles; ids differ by their uniforms
    base = synth.zipf_profile_logits(n_kinds, V, 1.1, 1.5, rng, "f32", rng.permutation(V))
    base[1::3] = rng.standard_normal((base[1::3].shape[0], V)) * 1.2   # nuclei wider than the candidate list
    base[4] = np.round(base[4] * 4) / 4                                # ties at every cut
    kind = np.arange(B) % n_kinds
    logits = synth.f32_to_bf16_bits(base) if dtype == "bf16" else base
    lens = np.where(kind % 2 == 0, 0, rng.integers(1, 2500, B))
    head = np.argpartition(-base, 4000, axis=1)[:, :4000]
    hist_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    hist_ids = np.concatenate([rng.choice(head[kind[b]], int(lens[b])) for b in range(B)]).astype(np.int32)
    params = synth.make_params(
        B, temperature=np.array([1.0, 1.1, 0.0, 0.8, 0.9, 1.0, 1.0, 1.0, 1.3, 0.7], np.float32)[kind],
        top_k=np.array([0, 0, 0, 50, 0, 1000, 0, 5000, 20_000, 0], np.int32)[kind],
        top_p=np.array([0.95, 0.9, 1.0, 0.9, 0.99, 0.97, 1.0, 1.0, 1.0, 0.9], np.float32)[kind],
        min_p=np.array([0, 0, 0, 0, 0, 0, 1e-4, 0, 0, 0.02], np.float32)[kind],
        rep_penalty=1.1, freq_penalty=0.2, pres_penalty=0.1, n_prompt=100)
    hot = np.sort(rng.choice(V, int(V * hot_share), replace=False)).astype(np.int32) if hot_share else None
    w = synth.Workload(f"large-{dtype}-{V}", B, V, dtype, logits[kind] if B < 100 else logits, params, hist_ptr, hist_ids, hot_ids=hot)
    src = torch.from_numpy(logits if dtype == "f32" else logits.view(np.int16)).cuda()
    src = src if dtype == "f32" else src.view(torch.bfloat16)
    if B >= 100:  # the batch is gathered on the GPU; the oracle reads the rows it is asked for
        full = src[torch.from_numpy(kind).cuda()].contiguous()
        dev = P.to_device(synth.Workload(w.name, B, V, dtype, logits, params, hist_ptr, hist_ids, hot_ids=hot))
        dev["logits"] = full
        rows = sorted(rng.choice(B, 20, replace=False).tolist())
        ids, dg = P.run_gpu(w, 1, dev=dev)
        one = []
        for r in rows:
            h = hist_ids[hist_ptr[r]:hist_ptr[r + 1]]
            wr = synth.Workload(w.name, 1, V, dtype, logits[kind[r]][None], params[r:r + 1], np.array([0, h.size]), h, hot_ids=hot)
            one += P.run_oracle(wr, 1, row_offset=r)
        P.compare(ids, dg, one, rows)
    else:
        for step in (0, 1):
            ids, dg = P.run_gpu(w, step)
            P.compare(ids, dg, P.run_oracle(w, step), range(B))
    flags = dg["flags"]
    assert not (flags & binding.DIAG_ERROR).any()
    if V >= 1 << 19:
        assert not (flags & binding.DIAG_GENERAL).any()  # (says that another kernel handed the row on)
        return
    # the routes complete their rows: nuclei wider than the list and top-k above it, the pattern counts of rows without
    # penalties and top-k; the general kernel is left the rows with thousands of ties at a cut and a few that miss
    handed = (flags & binding.DIAG_GENERAL) > 0
    assert handed[kind != 4].mean() <= 0.1, np.bincount(kind[handed], minlength=n_kinds)
    assert ((flags & binding.DIAG_WIDE) > 0)[np.isin(kind, (1, 7))].all()
    if dtype == "bf16":
        assert ((flags & binding.DIAG_PATTERN) > 0)[kind == 0].all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_handed_to_the_general_kernel_say_so(dtype):
    """Top-k under penalties that raise logits is the general kernel's at every size."""
    rng = np.random.default_rng(3)
    B, V = 4, 1 << 18
    z = rng.standard_normal((B, V)).astype(np.float32)
    w = synth.Workload("handed-on", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z,
                       synth.make_params(B, temperature=1.0, top_k=20, rep_penalty=np.array([1.1, 0.8, 1.1, 0.8], np.float32), n_prompt=5),
                       np.arange(B + 1, dtype=np.int64) * 10, rng.integers(0, V, B * 10).astype(np.int32))
    ids, dg = P.run_gpu(w, 0)
    P.compare(ids, dg, P.run_oracle(w, 0), range(B))
    assert (((dg["flags"] & binding.DIAG_GENERAL) > 0) == [False, True, False, True]).all()
