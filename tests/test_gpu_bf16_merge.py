"""The uncompressed decode step on both sides of the line between one launch and two (partials per item: 48; up to 16 MiB of
rows 64, at four query heads per KV head 96; 64 chunks), against attention in fp64: one and many chunks, sequences without rows, output memory that holds anything, the query's
own memory as output, and calls one after the other."""
import numpy as np
import pytest
import torch

from test_gpu_parity import B

pytestmark = pytest.mark.gpu


def _inputs(lens, hkv, g, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    K, V = (torch.randn(sum(lens) * hkv * 128, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    return K, V, torch.randn((len(lens), hkv * g, 128), generator=gen, device="cuda", dtype=torch.bfloat16)


def _exact(lens, hkv, g, K, V, q):
    out, lse, at = np.zeros((len(lens), hkv * g, 128)), np.full((len(lens), hkv * g), -np.inf), 0
    for s, T in enumerate(lens):
        n = hkv * T * 128
        k, v = (x[at:at + n].double().cpu().numpy().reshape(hkv, T, 128) for x in (K, V))
        at += n
        if T == 0:
            continue
        x = np.einsum("hgd,htd->hgt", q[s].double().cpu().numpy().reshape(hkv, g, 128), k) / np.sqrt(128.0)
        m = x.max(-1, keepdims=True)
        p = np.exp(x - m)
        l = p.sum(-1, keepdims=True)
        out[s] = np.einsum("hgt,htd->hgd", p / l, v).reshape(hkv * g, 128)
        lse[s] = (m + np.log(l)).reshape(-1)
    return out, lse


def _check(got, ref):
    out, lse = (x.double().cpu().numpy() for x in got)
    # probabilities as two bf16 terms (2^-16) and fp32 sums over at most 16K terms: 1e-4 of the largest component
    assert np.abs(out - ref[0]).max() <= 1e-4 * max(np.abs(ref[0]).max(), 1e-30)
    some = np.isfinite(ref[1])
    assert np.array_equal(np.isfinite(lse), some) and np.abs(lse[some] - ref[1][some]).max(initial=0.0) <= 1e-4


@pytest.mark.parametrize("lens,hkv,g", [
    ((1,), 2, 4), ((256,), 1, 1), ((257,), 2, 8), ((6 * 256,), 2, 8), ((8 * 256,), 8, 8), ((8 * 256 + 1,), 2, 8),
    ((4096,), 8, 4), ((4097,), 8, 4), ((24 * 256,), 2, 4), ((24 * 256 + 1,), 2, 4), ((64 * 256,), 2, 1), ((64 * 256 + 1,), 1, 1),
    ((32 * 256,), 2, 2), ((33 * 256 - 1,), 2, 2),
    ((0, 300, 0, 1), 2, 4), ((0, 9000), 8, 4), (tuple(range(1, 67)), 2, 2)])
def test_one_launch_and_two(lens, hkv, g):
    b = B()
    print(f"[case] lens {lens[:4]} hkv {hkv} g {g}", flush=True)
    K, V, q = _inputs(lens, hkv, g, sum(lens) + g)
    ref = _exact(lens, hkv, g, K, V, q)
    ws = torch.full((max(16, b.rdkv_decode_bf16_workspace_bytes(list(lens), hkv * g, hkv)),), 0xFF, device="cuda", dtype=torch.uint8)
    first = None
    for fill in (0, -1, 0x7FC00000):
        out = torch.full(q.shape, fill, device="cuda", dtype=torch.int32).view(torch.float32)
        lse = torch.full(q.shape[:-1], fill, device="cuda", dtype=torch.int32).view(torch.float32)
        for _ in range(3):               # the workspace and the output as the call before left them
            b.rdkv_decode_attn_bf16(K, V, list(lens), hkv * g, hkv, q, out=out, lse=lse, workspace=ws)
            got = out.clone(), lse.clone()
            _check(got, ref)
            first = first or got
            assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1])


def test_query_in_the_outputs_memory():
    b, lens, hkv, g = B(), (700, 1000), 2, 4
    K, V, q = _inputs(lens, hkv, g, 9)
    ref = _exact(lens, hkv, g, K, V, q)
    out = torch.zeros(q.shape, device="cuda", dtype=torch.float32)
    inside = out.view(torch.bfloat16).reshape(-1)[-q.numel():].view(q.shape)
    inside.copy_(q)
    _check(b.rdkv_decode_attn_bf16(K, V, list(lens), hkv * g, hkv, inside, out=out), ref)


# The outputs in an input's memory, with more workgroups than the chip holds: nothing is written there before all of it is read.
@pytest.mark.parametrize("lens,hkv,g", [((3000,) * 16, 8, 4), ((0, 300, 700), 2, 4)])
@pytest.mark.parametrize("what,where,end", [("lse", "q", False), ("lse", "q", True), ("lse", "K", False), ("lse", "V", True), ("out", "q", True),
                                            ("out", "K", False), ("out", "V", True)])
def test_outputs_in_an_inputs_memory(lens, hkv, g, what, where, end):
    b = B()
    print(f"[case] {what} in {where}, {len(lens)} sequences", flush=True)
    K, V, q = _inputs(lens, hkv, g, 11)
    ref = _exact(lens, hkv, g, K, V, q)
    n = q.numel() if what == "out" else q.shape[0] * q.shape[1]
    home = torch.zeros(max(4 * n, 2 * {"q": q, "K": K, "V": V}[where].numel()), device="cuda", dtype=torch.uint8)
    put = home.view(torch.bfloat16)
    args = {"q": q, "K": K, "V": V}
    x = args[where]
    inside = put[put.numel() - x.numel():] if end else put[:x.numel()]
    inside.copy_(x.reshape(-1))
    args[where] = inside.view(x.shape)
    shared = home.view(torch.float32)
    shared = shared[shared.numel() - n:] if end else shared[:n]
    outs = {what: shared.view(q.shape if what == "out" else q.shape[:-1])}
    got = b.rdkv_decode_attn_bf16(args["K"], args["V"], list(lens), hkv * g, hkv, args["q"], **outs)
    _check(got, ref)
