"""The library launches on the stream it is given, never synchronizes, and its launches can be
captured into a HIP graph (the benchmark's timed region is one); every replay must reproduce the
eager results bit for bit, including the work-balanced launches that pass partial sums through the
workspace."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_2410_16144_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def ops():
    from paper_2410_16144_amd import binding
    from paper_2410_16144_amd import ops as _ops
    binding.lib()
    return _ops


def _layers(ops, dev, count, hidden, ffn, M):
    from paper_2410_16144_amd.decode_layer import make_layer
    return [make_layer(2, 50 + i, hidden, ffn, M, dev, 0.4, 0.01)[0] for i in range(count)]


def _snapshot(layers):
    return [[o.clone() for o in l.outs] for l in layers]


def _same(a, b):
    return all(torch.equal(x, y) for la, lb in zip(a, b) for x, y in zip(la, lb))


@pytest.mark.parametrize("M", [1, 4])
def test_graph_replays_equal_eager(dev, ops, M):
    layers = _layers(ops, dev, 3, 3200, 8640, M)     # M = 1 takes the work-balanced kernel (workspace)
    for l in layers:
        l.step_fused()
    torch.cuda.synchronize()
    ref_fused = _snapshot(layers)
    for l in layers:
        l.step_single_launch()
    torch.cuda.synchronize()
    assert _same(ref_fused, _snapshot(layers))
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            for l in layers:
                l.step_fused()
            for l in layers:
                l.step_single_launch()
    torch.cuda.synchronize()
    for replay in range(4):
        for l in layers:
            for o in l.outs:
                o.fill_(float(replay))          # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert _same(ref_fused, _snapshot(layers)), "replay %d" % replay
    assert not ops.workspace(dev).any()


def test_launches_follow_the_given_stream(dev, ops):
    """A long kernel is queued on a side stream first; the products queued behind it on the same stream
    must see its result, which they only do if they really run on that stream."""
    rng = synth.rng_for(4242)
    K, N, M = 2048, 512, 2
    w = synth.ternary_weights(rng, N, K)
    bits = synth.to_bf16_bits(synth.activations(rng, M, K))
    pw = ops.pack_ternary(torch.from_numpy(w).to(dev), 0.02)
    x_final = torch.from_numpy(bits.view(np.int16)).to(dev).view(torch.bfloat16)
    x = torch.zeros_like(x_final)
    big = torch.empty(1 << 28, dtype=torch.uint8, device=dev)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(8):
            big.fill_(1)                       # a few hundred microseconds of work ahead in the queue
        x.copy_(x_final)                       # the product's input only becomes valid after it
        qa = ops.quant_act(x)
        out, acc = ops.gemv(pw, qa, want_acc=True)
        out2, acc2 = ops.gemm(pw, qa, want_acc=True)
        grp = ops.DecodeGroup([pw], [x], want_acc=True)
        grp.launch()
    side.synchronize()
    q_ref, a_ref, _ = oracle.quant_act(bits)
    acc_ref = oracle.matmul_i32(q_ref, w)
    for got in (acc, acc2, grp.accs[0]):
        assert np.array_equal(got.cpu().numpy(), acc_ref)
    assert torch.equal(out, out2) and torch.equal(out, grp.outs[0])


COLD = r"""
import sys
import torch
from paper_2410_16144_amd import binding as B, decoder, ops
dev = torch.device("cuda")


def captured_first(what, call, out):
    # a capture of the kernel's first use in this process; three replays against the eager call that follows
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            call()
    got = []
    for _ in range(3):
        out.fill_(-7.0)
        g.replay()
        got.append(out.clone())
    out.fill_(-7.0)
    call()
    torch.cuda.synchronize()
    assert bool((out != -7.0).any()) and all(torch.equal(t, out) for t in got), what
    print(what, B.bl_last_kernel(), flush=True)


stream = lambda: torch.cuda.current_stream().cuda_stream
for d in (8, 36, 96, 128, 256):
    heads, pos0, M = 2, 40, 70
    q, k, v = (torch.randn(M, heads * d, device=dev) for _ in range(3))
    kc, vc = (torch.randn(pos0 + M, heads * d, device=dev).bfloat16() for _ in range(2))
    table, out = decoder.rope_table(d, pos0 + M, dev), torch.empty_like(q)
    scratch = torch.zeros(B.bl_attn_prefill_scratch_bytes(heads, d, pos0, M), dtype=torch.uint8, device=dev)
    captured_first("prompt attention %d" % d, lambda: B.bl_attn_prefill(
        q.data_ptr(), k.data_ptr(), v.data_ptr(), table.data_ptr(), kc.data_ptr(), vc.data_ptr(), out.data_ptr(), scratch.data_ptr(),
        heads, d, pos0 + M, pos0, M, stream()), out)
pw = ops.pack_ternary(torch.randint(-1, 2, (300, 1000), dtype=torch.int8, device=dev), 0.02)
for M, form in ((9, 0), (40, 1016), (40, 1032), (40, 2016), (40, 2032), (40, 4032), (70, 4064), (70, 12), (70, 14), (70, 22), (70, 23),
                (70, 24), (70, 122), (70, 124), (70, 40022), (70, 40021), (70, 60021), (70, 40121), (70, 40012), (70, 30024), (70, 30023)):
    qa = ops.alloc_quant(M, 1000, dev)
    qa.q.random_(-127, 128)
    qa.a_scale.fill_(0.01)
    qa.q_sum.copy_(qa.q.sum(1, dtype=torch.int32))
    out = torch.empty(M, 300, device=dev)
    B.bl_set_tuning("gemm_mb", form)
    captured_first("gemm %d" % form, lambda: ops.gemm(pw, qa, out=out), out)
B.bl_set_tuning("gemm_mb", 25)
pw = ops.pack_ternary(torch.randint(-1, 2, (11008, 128), dtype=torch.int8, device=dev), 0.02)
qa = ops.alloc_quant(512, 128, dev)
qa.q.random_(-127, 128)
qa.a_scale.fill_(0.01)
qa.q_sum.copy_(qa.q.sum(1, dtype=torch.int32))
out = torch.empty(512, 11008, device=dev)
captured_first("gemm 25", lambda: ops.gemm(pw, qa, out=out), out)
assert "mixed_pair_gemm_kernel" in B.bl_last_kernel()
x, y, gamma = torch.randn(3, 5000, device=dev), torch.empty(3, 5000, device=dev), torch.rand(5000, device=dev)
captured_first("norm", lambda: decoder.norm_quant(B.BL_NORM_PLAIN, gamma, a=x, y=y, quantize=False), y)
print("all of them")
"""


def test_a_kernels_first_use_may_be_a_captured_one(dev):
    """Prompt attention, every form of the prefill product and the norm, each captured in a process that has not run it."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", COLD], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "all of them" in r.stdout, r.stdout[-1500:] + r.stderr[-1500:]
