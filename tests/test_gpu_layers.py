"""The per-token loop over several routed layers (Section 3.2.1: routing in the latter half of the layers; Section
3.4.2: per layer routing keys in device memory, pooled content bank in device or host memory): three layers with
their own banks and queries chained through paper_2603_23516_amd.layers.LayerStack, every layer's selection and
attention output against the oracle, with the pooled banks in HBM and in pinned host memory, on one stream and with
routing overlapped with fetch + attention on two streams."""
import numpy as np
import pytest
import torch

import msa_synth as S
import paper_2603_23516_amd as msa
from msa_synth import device as SD
from oracle import msa_oracle as O
from paper_2603_23516_amd.layers import LayerStack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tier", ["hbm", "host"])
def test_three_routed_layers_against_the_oracle(tier):
    L, N, Hkv, r, G, d, P, B, M, k, Lloc, base = 3, 90, 2, 4, 256, 128, 32, 3, 1, 5, 40, 1e6
    print(f"3 routed layers, pooled banks in {tier}: N={N} Hkv={Hkv} r={r} G={G} P={P} B={B} k={k} Lloc={Lloc}", flush=True)
    Hq, C = Hkv * r, G // P
    cfg = msa.MsaConfig(N, G, P, Hq, Hkv, d, base)
    stack = LayerStack(cfg, L, B, M, k, Lloc, tier=tier)
    host = []
    qs, Kls, Vls = [], [], []
    for l in range(L):
        sd = 95000 + 10 * l
        Kb, K = S.normal_bf16(sd, (N, Hkv, G, d))
        Vb, V = S.normal_bf16(sd + 1, (N, Hkv, G, d))
        qb, q = S.normal_bf16(sd + 2, (B, M, Hq, d))
        Klb, Kl = S.normal_bf16(sd + 3, (B, Hkv, Lloc, d))
        Vlb, Vl = S.normal_bf16(sd + 4, (B, Hkv, Lloc, d))
        host.append((K, V, q, Kl, Vl))
        buf = SD.bits_to_torch(Kb)                        # one staging buffer per layer: keys, then values
        stack.set_layer_keys(l, buf)
        buf.copy_(SD.bits_to_torch(Vb))
        stack.set_layer_values(l, buf)
        qs.append(SD.bits_to_torch(qb))
        Kls.append(SD.bits_to_torch(Klb))
        Vls.append(SD.bits_to_torch(Vlb))
    torch.cuda.synchronize()
    pos0 = k                                              # Section 3.2.2: local positions start at k
    q_pos = np.full((B, M), pos0 + Lloc - 1)
    dpos = torch.from_numpy(q_pos.astype(np.int32)).cuda()
    results = {}
    for overlap in (False, True, True):
        outs = [torch.zeros_like(qs[0]) for _ in range(L)]
        lses = [torch.zeros((B, M, Hq), dtype=torch.float32, device="cuda") for _ in range(L)]
        stack.step(qs, Kls, Vls, pos0, dpos, outs, lses, overlap=overlap)
        torch.cuda.synchronize()
        results[overlap] = ([o.clone() for o in outs], [x.clone() for x in lses], [i.clone() for i in stack.idx])
    for a, b in zip(results[False][0] + results[False][1] + results[False][2],
                    results[True][0] + results[True][1] + results[True][2]):
        assert torch.equal(a.view(torch.int32) if a.dtype == torch.float32 else a.view(torch.int16) if a.dtype == torch.bfloat16 else a,
                           b.view(torch.int32) if b.dtype == torch.float32 else b.view(torch.int16) if b.dtype == torch.bfloat16 else b)
    outs, lses, idxs = results[True]
    for l, (K, V, q, Kl, Vl) in enumerate(host):
        KRb, _ = O.routing_keys(K, P)
        oi, ov, _ = O.score_topk(q, KRb, C, k)
        assert np.array_equal(idxs[l].cpu().numpy(), oi), f"layer {l}: selection"
        Kbar = O.bf16_round(O.pool_rotated_keys(K, P, base))
        Vbar = O.bf16_round(O.pool_values(V, P))
        oo, ol = O.sparse_attend(q, Kbar, Vbar, oi, Kl, Vl, pos0, q_pos, base, mem_rotated=True)
        go = outs[l].float().cpu().numpy().astype(np.float64)
        gl = lses[l].cpu().numpy().astype(np.float64)
        err = np.abs(go - oo)
        rel = np.linalg.norm(err) / np.linalg.norm(oo)
        print(f"   layer {l}: max-abs {err.max():.3e} rel-L2 {rel:.3e}", flush=True)
        assert err.max() <= 2e-2 and rel <= 5e-3
        assert np.allclose(gl, ol, rtol=0, atol=5e-3)
    index_bytes, bank_bytes = stack.bytes()
    assert index_bytes == L * (msa.routing_keys_bytes(cfg) + msa.inv_norm_bytes(cfg))
    assert bank_bytes == L * 2 * N * Hkv * C * d * 2


@pytest.mark.parametrize("L,N,B", [(2, 8192, 3), (2, 8193, 3), (3, 7813, 9), (3, 7811, 1), (2, 8195, 17)])
def test_layers_whose_indexes_outgrow_the_cache(L, N, B):
    """Layers of 128 MB each, together just under and just over 256 MB, below and above 128 MB: selections and scores are bit for
    bit those of a call of its own, streaming loads or plain."""
    G, P, Hkv, d, k, Lloc = 64, 8, 8, 128, 9, 16
    print(f"{L} routed layers of {N} documents, {B} queries", flush=True)
    cfg = msa.MsaConfig(N, G, P, Hkv, Hkv, d, 1e4)
    stack = LayerStack(cfg, L, B, 1, k, Lloc)
    gen = torch.Generator("cuda").manual_seed(97000 + N)
    for l in range(L):
        bank = torch.randn((N, Hkv, G, d), generator=gen, device="cuda", dtype=torch.bfloat16)
        stack.set_layer_keys(l, bank)
        stack.set_layer_values(l, bank)
    del bank
    qs = [torch.randn((B, 1, Hkv, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(L)]
    loc = [torch.randn((B, Hkv, Lloc, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(L)]
    dpos = torch.full((B, 1), k + Lloc - 1, dtype=torch.int32, device="cuda")
    for overlap in (False, True):
        stack.step(qs, loc, loc, k, dpos, [None] * L, [None] * L, overlap=overlap)
        torch.cuda.synchronize()
        for l in range(L):
            idx, val = msa.msa_score_topk(cfg, qs[l], stack.KR[l], stack.inv[l], k)
            torch.cuda.synchronize()
            assert torch.equal(idx, stack.idx[l]) and torch.equal(val.view(torch.int32), stack.val[l].view(torch.int32))


def test_refused_layer_leaves_nothing_behind():
    """A step with one layer that attention refuses raises before anything runs; the next step is whole, on one stream, on
    two, and without outputs that are not wanted."""
    L, N, Hkv, r, G, d, P, B, k, Lloc = 3, 60, 2, 2, 128, 64, 32, 2, 4, 33
    Hq = Hkv * r
    stack = LayerStack(msa.MsaConfig(N, G, P, Hq, Hkv, d, 1e4), L, B, 1, k, Lloc)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(97000)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    for l in range(L):
        stack.set_layer_keys(l, rnd(N, Hkv, G, d))
        stack.set_layer_values(l, rnd(N, Hkv, G, d))
    qs, Kls, Vls = ([rnd(*s) for _ in range(L)] for s in ((B, 1, Hq, d), (B, Hkv, Lloc, d), (B, Hkv, Lloc, d)))
    pos = torch.full((B, 1), k + Lloc - 1, dtype=torch.int32, device="cuda")
    odd = torch.zeros(Kls[0].numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(B, Hkv, Lloc, d)   # not 16-byte aligned
    runs = []
    for overlap in (True, False):
        outs = [torch.full_like(q, 7.0) for q in qs]
        lses = [torch.full((B, 1, Hq), 7.0, device="cuda") for _ in range(L)]
        for i in stack.idx:
            i.fill_(-7)
        for at in range(L):
            bad = [odd if l == at else x for l, x in enumerate(Kls)]
            with pytest.raises(msa.MsaError) as e:
                stack.step(qs, bad, Vls, k, pos, outs, lses, overlap=overlap)
            assert e.value.status == msa.MSA_ERR_MISALIGNED
        torch.cuda.synchronize()
        assert all(bool((o == 7.0).all()) for o in outs + lses) and all(bool((i == -7).all()) for i in stack.idx)
        stack.step(qs, Kls, Vls, k, pos, outs, lses, overlap=overlap)
        torch.cuda.synchronize()
        runs.append([t.clone() for t in outs + lses + stack.idx])
        assert all(bool((i >= 0).all()) for i in stack.idx)
        part = [torch.full_like(qs[0], 7.0)] + [None] * (L - 1)
        stack.step(qs, Kls, Vls, k, pos, part, [None] * L, overlap=overlap)
        torch.cuda.synchronize()
        assert torch.equal(part[0].view(torch.int16), outs[0].view(torch.int16))
    for a, b in zip(*runs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("two", [False, True])
def test_steps_from_several_streams_and_a_graph(two):
    """Steps called on two streams in turn share the stack's workspaces: they follow each other, with attention beside the
    next layer's routing or not; and a captured step replays with eager steps between its replays."""
    L, N, Hkv, r, G, d, P, B, k, Lloc = 3, 3000, 4, 2, 256, 64, 32, 6, 8, 70
    Hq = Hkv * r
    stack = LayerStack(msa.MsaConfig(N, G, P, Hq, Hkv, d, 1e4), L, B, 1, k, Lloc)
    assert not stack.two_streams
    stack.two_streams = two
    gen = torch.Generator(device="cuda")
    gen.manual_seed(98000)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    for l in range(L):
        stack.set_layer_keys(l, rnd(N, Hkv, G, d))
        stack.set_layer_values(l, rnd(N, Hkv, G, d))
    Kls, Vls = ([rnd(B, Hkv, Lloc, d) for _ in range(L)] for _ in range(2))
    pos = torch.full((B, 1), k + Lloc - 1, dtype=torch.int32, device="cuda")
    batches = [[rnd(B, 1, Hq, d) for _ in range(L)] for _ in range(6)]

    def buffers():
        return [torch.zeros(B, 1, Hq, d, dtype=torch.bfloat16, device="cuda") for _ in range(L)]
    lses = [None] * L
    want = []
    for qs in batches:
        outs = buffers()
        stack.step(qs, Kls, Vls, k, pos, outs, lses, overlap=False)
        torch.cuda.synchronize()
        want.append(outs)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [buffers() for _ in batches]
    torch.cuda.synchronize()
    for i, qs in enumerate(batches):
        with torch.cuda.stream(streams[i % 2]):
            stack.step(qs, Kls, Vls, k, pos, got[i], lses)
    torch.cuda.synchronize()
    for x, y in zip(want, got):
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(x, y))
    fixed, outs = [q.clone() for q in batches[0]], buffers()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        stack.step(fixed, Kls, Vls, k, pos, outs, lses)
    for i in (3, 1, 5):
        for a, b in zip(fixed, batches[i]):
            a.copy_(b)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(outs, want[i]))
        eager = buffers()
        stack.step(batches[2], Kls, Vls, k, pos, eager, lses)
        torch.cuda.synchronize()
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(eager, want[2]))


def small_stack(two):
    L, N, Hkv, r, G, d, P, B, k, Lloc = 2, 500, 2, 2, 64, 64, 32, 3, 4, 40
    stack = LayerStack(msa.MsaConfig(N, G, P, Hkv * r, Hkv, d, 1e4), L, B, 1, k, Lloc)
    stack.two_streams = two
    gen = torch.Generator(device="cuda")
    gen.manual_seed(98500)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    for l in range(L):
        stack.set_layer_keys(l, rnd(N, Hkv, G, d))
        stack.set_layer_values(l, rnd(N, Hkv, G, d))
    qs, Kls, Vls = ([rnd(*x) for _ in range(L)] for x in ((B, 1, Hkv * r, d), (B, Hkv, Lloc, d), (B, Hkv, Lloc, d)))
    outs = [torch.zeros_like(q) for q in qs]
    args = (qs, Kls, Vls, k, torch.full((B, 1), k + Lloc - 1, dtype=torch.int32, device="cuda"), outs, [None] * L)
    torch.cuda.synchronize()
    return stack, args


def apart(n):
    """A stream and n more whose work it does not hold up (streams share a few hardware queues)."""
    x = torch.zeros(1, device="cuda")
    first, others = torch.cuda.Stream(), []
    for other in [torch.cuda.Stream() for _ in range(12)]:
        torch.cuda.synchronize()
        with torch.cuda.stream(first):
            torch.cuda._sleep(200_000_000)
        with torch.cuda.stream(other):
            x.add_(1)
        other.synchronize()
        if not first.query():
            others.append(other)
        torch.cuda.synchronize()
        if len(others) == n:
            return first, others
    pytest.skip("no streams run beside each other here")


@pytest.mark.parametrize("two", [False, True])
def test_step_waits_for_the_step_before_alone(two):
    """Work that a caller put on its stream behind a step does not hold up the next step from another stream."""
    stack, args = small_stack(two)
    first, (other, stack.s_attend) = apart(2)
    stack.step(*args)
    torch.cuda.synchronize()
    want = [o.clone() for o in args[5]]
    with torch.cuda.stream(first):
        stack.step(*args)
        torch.cuda._sleep(1_000_000_000)   # half a second
    with torch.cuda.stream(other):
        stack.step(*args)
    other.synchronize()
    assert not first.query()
    torch.cuda.synchronize()
    assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(want, args[5]))


def test_step_after_its_last_stream_was_destroyed():
    """The stack keeps no stream of its callers: one that its owner has destroyed is not touched again."""
    import ctypes
    loaded = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
    assert len(loaded) == 1
    hip = ctypes.CDLL(loaded.pop())   # the runtime that torch uses, not another copy of it
    stack, args = small_stack(False)
    stack.step(*args)
    torch.cuda.synchronize()
    want = [o.clone() for o in args[5]]
    for _ in range(3):
        handle = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(handle)) == 0
        with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
            stack.step(*args)
        torch.cuda.synchronize()
        assert hip.hipStreamDestroy(handle) == 0
        assert not any(isinstance(v, torch.cuda.Stream) and v.cuda_stream == handle.value for v in vars(stack).values())
        stack.step(*args)
        torch.cuda.synchronize()
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(want, args[5]))
