"""msa_score_topk_noalloc (the entry point for callers that cannot allocate: it runs on a scratch buffer built
into the library) against msa_score_topk with a caller's workspace: the same kernels, so bit-identical
selections and scores.  Two calls in a row on the shared buffer, the second with a smaller input, each compared
with the existing entry point and, for the selection, with the oracle."""
import numpy as np
import pytest
import torch

import msa_synth as S
import paper_2603_23516_amd as msa
from msa_synth import device as SD
from oracle import msa_oracle as O

pytestmark = pytest.mark.gpu


def _case(N, Hkv, r, G, d, P, B, M, k, seed):
    cfg = msa.MsaConfig(N, G, P, Hkv * r, Hkv, d, 1e4)
    Kb, K = S.normal_bf16(S.seed_for(9, seed), (N, Hkv, G, d))
    qb, q = S.normal_bf16(S.seed_for(9, seed + 1), (B, M, Hkv * r, d))
    dK, dq = SD.bits_to_torch(Kb), SD.bits_to_torch(qb)
    KR, inv = msa.msa_build_routing_keys(cfg, dK)
    torch.cuda.synchronize()
    return cfg, K, q, dq, KR, inv


def _run_both(cfg, dq, KR, inv, k):
    B, M = dq.shape[0], dq.shape[1]
    ref_idx, ref_val = msa.msa_score_topk(cfg, dq, KR, inv, k)
    torch.cuda.synchronize()
    idx = torch.full_like(ref_idx, -7)
    val = torch.full_like(ref_val, float("nan"))
    before = torch.cuda.memory_allocated()
    print(f"msa_score_topk_noalloc N={cfg.n_docs} B={B} M={M} k={k}", flush=True)
    msa.msa_score_topk_noalloc(cfg, dq, KR, inv, k, idx, val)
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    assert torch.equal(idx, ref_idx)
    assert torch.equal(val, ref_val)
    return idx.cpu().numpy(), val.cpu().numpy()


def test_noalloc_matches_workspace_entry_point_twice():
    # first call: several tiles per wave, ragged last tile (N * C = 1000 * 8 keys, 500 tiles), 3 queries
    cfg1, K1, q1, dq1, KR1, inv1 = _case(N=1000, Hkv=2, r=4, G=512, d=64, P=64, B=3, M=1, k=8, seed=10)
    gi1, gv1 = _run_both(cfg1, dq1, KR1, inv1, 8)
    # second call, right after, smaller input (its buffers lie inside what the first call left behind)
    cfg2, K2, q2, dq2, KR2, inv2 = _case(N=37, Hkv=2, r=4, G=512, d=64, P=64, B=1, M=1, k=4, seed=20)
    gi2, gv2 = _run_both(cfg2, dq2, KR2, inv2, 4)
    # and the first again: the buffer now holds the second call's leftovers
    gi1b, gv1b = _run_both(cfg1, dq1, KR1, inv1, 8)
    assert np.array_equal(gi1, gi1b) and np.array_equal(gv1, gv1b)
    # the selections are the oracle's (random scores: no ties at this size)
    for (K, q, cfg, k, gi, gv) in ((K1, q1, cfg1, 8, gi1, gv1), (K2, q2, cfg2, 4, gi2, gv2)):
        KRb, _ = O.routing_keys(K, cfg.chunk)
        oi, ov, _ = O.score_topk(q, KRb, cfg.chunks_per_doc, k)
        assert np.array_equal(gi, oi)
        assert np.allclose(gv, ov, rtol=0, atol=2e-5)


def test_noalloc_refuses_what_does_not_fit():
    cfg = msa.MsaConfig(65536, 512, 64, 32, 8, 128, 1e6)
    assert msa.score_topk_workspace_bytes(cfg, 1, 8192, 8) > msa.noalloc_scratch_bytes()
    q = torch.zeros((1, 8192, 32, 128), dtype=torch.bfloat16, device="cuda")
    KR, inv = msa.alloc_routing_index(cfg)
    idx = torch.empty((1, 8192, 8, 8), dtype=torch.int32, device="cuda")
    with pytest.raises(msa.MsaError) as e:
        msa.msa_score_topk_noalloc(cfg, q, KR, inv, 8, idx, None)
    assert e.value.status == msa.MSA_ERR_WORKSPACE
