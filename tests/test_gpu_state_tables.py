"""The tables of an incremental penalty state, where their groups of eight entries and rounds of 256 groups end: sequences that are
restarted (few at a time, or more than there are compute units) and get chosen ids appended sample as the call that is handed the
same token lists: same ids, same masses (which every count and every mask bit enters)."""
import numpy as np
import pytest

from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,B,n0", [(9_000, 6, 0), (9_024, 300, 7), (33_000, 256, 130), (33_000, 257, 130), (140_033, 6, 2040), (140_000, 4, 4600),
                                    (262_143, 4, 9_000), (300_000, 3, 20)])
def test_restarted_and_appended(V, B, n0):
    import torch
    rng = np.random.default_rng(V + B)
    steps, L_max = 20, n0 + 20
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    rows = [rng.choice(V, size=max(n0 - b % 9, 0), replace=b % 2 == 1).astype(np.int32) for b in range(B)]
    half = np.array([r.size // 2 for r in rows], np.int32)
    csr = lambda: (dev(np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)), dev(np.concatenate(rows + [np.zeros(1, np.int32)])))
    params = synth.make_params(B, temperature=1.0, rep_penalty=1.2, freq_penalty=0.3, pres_penalty=0.1)
    params["n_prompt"] = half
    params["top_k"][::3] = 40
    par = dev(params.view(np.uint8).reshape(B, 32))
    lg = torch.randn(B, V, generator=torch.Generator(device="cuda:0").manual_seed(V), device="cuda:0")
    s = binding.Sampler(V, L_max, max_B=B)
    state = binding.simple_state_create(0, B, V, L_max)
    stream = torch.cuda.current_stream().cuda_stream
    ptr, ids = csr()
    half_d = dev(half)
    assert binding.simple_state_restart(state, 0, B, ptr.data_ptr(), ids.data_ptr(), half_d.data_ptr(), stream) == 0
    chosen = [0, V - 1, 1, 63, 64, 511, 512, 513, V - 2, V // 64 * 64 - 1, V // 2]
    for step in range(steps):
        if step % 4 == 0 or step == steps - 1:
            ptr, ids = csr()
            out, out_c = (torch.full((B,), -9, dtype=torch.int32, device="cuda:0") for _ in range(2))
            dg, dg_c = (torch.zeros(B * 32, dtype=torch.uint8, device="cuda:0") for _ in range(2))
            assert binding.simple_sample_state(s.ctx, state, 0, lg.data_ptr(), B, V, binding.SIMPLE_F32, V, par.data_ptr(), 0, 0, 11, step, 0,
                                               out.data_ptr(), dg.data_ptr(), stream) == 0
            s.sample(lg, par, ptr, ids, seed=11, step=step, out=out_c, diag=dg_c, V=V)
            torch.cuda.synchronize()
            assert torch.equal(out, out_c)
            d, d_c = (x.cpu().numpy().view(binding.ROW_DIAG_DTYPE) for x in (dg, dg_c))
            assert np.array_equal(d["s_k"], d_c["s_k"]) and np.array_equal(d["p_chosen"], d_c["p_chosen"]) and np.array_equal(d["flags"], d_c["flags"])
            assert not (d["flags"] & binding.DIAG_ERROR).any()
        # chosen ids, ids that the sequence has, and others
        new = np.array([chosen[(step + b) % len(chosen)] if (step + b) % 3 == 0 else
                        (int(rng.choice(rows[b])) if rows[b].size and (step + b) % 3 == 1 else int(rng.integers(V))) for b in range(B)], np.int32)
        new_d = dev(new)
        assert binding.simple_state_append(state, 0, new_d.data_ptr(), B, stream) == 0
        torch.cuda.synchronize()
        rows = [np.append(r, t).astype(np.int32) for r, t in zip(rows, new)]
    binding.simple_state_destroy(state)
    s.close()
