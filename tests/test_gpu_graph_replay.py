"""A captured sampling call can be replayed: every replay finds the row queues empty and leaves them
empty, whatever ran in between, so it returns the eager call's ids.  The batches hold rows for every
queue (sliced kernels, general kernel, the hot-first call's rejected tails), more of them over the
replays than a context has places."""
import numpy as np
import pytest

import parity_util as P
from paper_2512_00719_amd import binding, synth

pytestmark = pytest.mark.gpu

REPLAYS = 6


def _replays_match(call, between, B):
    """call(out) enqueues on the current stream; `between` is eager work on the same context."""
    import torch
    out = torch.full((B,), -9, dtype=torch.int32, device="cuda:0")
    want = torch.full((B,), -9, dtype=torch.int32, device="cuda:0")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(want)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    assert (want >= 0).all()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(out)
    for r in range(REPLAYS):
        out.fill_(-9)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), (r, (out != want).nonzero()[:8].flatten().tolist())
        for _ in range(r):  # an odd and an even number of other calls
            between()
    torch.cuda.synchronize()


def _mixed(B, V, dtype, offset=0):
    """Controls of every route, many rows of each queue: untruncated, wide nucleus, top-k above the list, raising penalties."""
    import torch
    rng = np.random.default_rng(V + B)
    z = synth.zipf_profile_logits(B, V, 1.1, 1.5, rng, "f32", rng.permutation(V))
    z[1::4] = rng.standard_normal((z[1::4].shape[0], V)) * 1.2
    n = min(300, V)
    hist_ptr = np.arange(B + 1, dtype=np.int64) * n
    hist_ids = rng.integers(0, V, B * n).astype(np.int32)
    params = synth.make_params(
        B, temperature=1.1, top_k=np.resize([0, 0, 40, 3000], B).astype(np.int32), top_p=np.resize([1.0, 0.97, 0.9, 0.99], B).astype(np.float32),
        rep_penalty=np.resize([1.1, 1.1, 0.8, 1.1], B).astype(np.float32), freq_penalty=0.2, pres_penalty=0.1, n_prompt=n // 2)
    w = synth.Workload("replay", B, V, dtype, synth.f32_to_bf16_bits(z) if dtype == "bf16" else z, params, hist_ptr, hist_ids)
    dev = P.to_device(w)
    if offset:
        buf = torch.zeros(B * V + 16, dtype=dev["logits"].dtype, device="cuda:0")
        buf[offset:offset + B * V] = dev["logits"].reshape(-1)
        dev["logits"] = buf[offset:offset + B * V].view(B, V)
    return w, dev


@pytest.mark.parametrize("V,dtype,offset,B", [(1000, "f32", 0, 40), (40_001, "f32", 1, 40), (40_960, "f32", 0, 300), (50_048, "bf16", 0, 40),
                                              (1 << 18, "bf16", 0, 12)])
def test_a_captured_call_replays(V, dtype, offset, B):
    w, dev = _mixed(B, V, dtype, offset)
    other, odev = _mixed(9, 30_000, "f32")
    s = binding.Sampler(max(V, 30_000), 300, max_B=max(B, 9))
    _replays_match(lambda out: s.sample(dev["logits"], dev["params"], dev["hist_ptr"], dev["hist_ids"], seed=w.seed, step=3, out=out, V=V),
                   lambda: s.sample(odev["logits"], odev["params"], odev["hist_ptr"], odev["hist_ids"], seed=1, step=1, V=30_000), B)
    s.close()


def test_a_captured_static_call_replays():
    import torch
    w, dev = _mixed(100, 40_000, "f32")  # two launches of the static entry point
    other, odev = _mixed(9, 30_000, "f32")

    def call(x, d, out):
        rc = binding.simple_sample_static(d["logits"].data_ptr(), x.B, x.V, binding.SIMPLE_F32, x.V, d["params"].data_ptr(), d["hist_ptr"].data_ptr(),
                                          d["hist_ids"].data_ptr(), 0, 0, x.seed, 3, 0, out.data_ptr(), 0, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
    scratch = torch.empty(9, dtype=torch.int32, device="cuda:0")
    _replays_match(lambda out: call(w, dev, out), lambda: call(other, odev, scratch), 100)


@pytest.mark.parametrize("dtype,H,B", [("f32", 1024, 24), ("bf16", 2048, 24)])
def test_a_captured_hot_first_call_replays(dtype, H, B):
    """Tails above what a row's own workgroup streams, as heavy as the hot set: most rows are queued."""
    import torch
    from test_gpu_hot_first import _dev, tail_stats
    V = H + 81_920
    rng = np.random.default_rng(H)
    z = rng.standard_normal((B, V)).astype(np.float32)
    bits = synth.f32_to_bf16_bits(z)
    if dtype == "bf16":
        z = synth.bf16_bits_to_f32(bits)
    params = synth.make_params(B, temperature=1.0)
    params["top_k"][::5] = 30  # and some for the general kernel
    lg = _dev(z if dtype == "f32" else bits.view(np.int16))
    ts, par = _dev(tail_stats(z, params, H).view(np.uint8).reshape(B, 16)), _dev(params.view(np.uint8).reshape(B, 32))
    s = binding.Sampler(V, 0, max_B=B)

    def call(step, out):
        rc = binding.simple_sample_hot_first(s.ctx, lg.data_ptr(), B, V, binding.SIMPLE_F32 if dtype == "f32" else binding.SIMPLE_BF16, V,
                                             par.data_ptr(), H, ts.data_ptr(), 5, step, 0, out.data_ptr(), 0, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
    scratch = torch.empty(B, dtype=torch.int32, device="cuda:0")
    _replays_match(lambda out: call(7, out), lambda: call(8, scratch), B)
    s.close()
