"""Branches of the work plans at the sizes where they can go wrong, against the float64 oracle (tolerances as in
test_gpu_parity.py)."""
import numpy as np
import pytest
import torch

import msa_synth as S
import paper_2603_23516_amd as msa
from oracle import msa_oracle as O

from test_gpu_parity import check_topk_generic, dev, say, upload_oracle_index

pytestmark = pytest.mark.gpu


def random_index(seed, N, Hkv, C, d):
    _, KRb = S.normal_bf16(seed, (Hkv, N * C, d))
    return KRb, 1.0 / np.maximum(np.linalg.norm(KRb, axis=-1), O.EPS_NORM)


def device_index(seed, Hkv, NC, d):
    """Random keys bf16 [Hkv][NC][d] on the device, and the same in the index's tiles."""
    tiles = (NC + 15) // 16
    keys = torch.randn((Hkv, tiles * 16, d), generator=torch.Generator("cuda").manual_seed(seed), device="cuda").to(torch.bfloat16)
    return keys[:, :NC], keys.reshape(Hkv, tiles, 16, d // 8, 8).transpose(2, 3).contiguous()


def call_us(cfg, q, KR, inv, k):
    """Outputs of msa_score_topk and the shortest of its calls."""
    ws = torch.empty(msa.score_topk_workspace_bytes(cfg, q.shape[0], q.shape[1], k), dtype=torch.uint8, device="cuda")
    idx, val = msa.msa_score_topk(cfg, q, KR, inv, k, workspace=ws)
    best = 1e9
    for _ in range(15):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        msa.msa_score_topk(cfg, q, KR, inv, k, idx, val, ws)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return idx, val, best


# (N, Hkv, r, C, d, B, M, k, sim): the all-heads scan writes a score matrix
ALL_SCAN = [
    (5, 8, 1, 8, 128, 1, 1, 5, "cos"),            # fewer tiles than one workgroup has waves
    (1037, 4, 2, 16, 128, 9, 1, 33, "cos"),       # 16-query pass, one document per tile
    (8193, 8, 1, 8, 128, 25, 1, 16, "cos"),       # 32-query pass, units of several tiles, ragged last tile
    (4099, 8, 2, 1, 64, 33, 1, 20, "dot"),        # one query more than the scan takes: the wide kernel
    (4099, 8, 2, 1, 64, 20, 1, 20, "dot"),        # no norms to read, sixteen documents per tile
    (16400, 2, 1, 2, 64, 2, 2, 64, "cos"),        # whole rows held by sixteen waves
    (12437, 8, 1, 8, 64, 5, 1, 64, "cos"),        # ... twelve documents per lane, as many winners as lanes in a wave
    (32768, 2, 1, 1, 64, 1, 1, 64, "cos"),        # the longest row that one workgroup takes
    (32785, 2, 1, 2, 64, 2, 2, 64, "cos"),        # rows in five parts, the last of 17 documents (fewer than k)
    (200007, 2, 1, 1, 64, 25, 1, 7, "cos"),       # two segments of the bank
    (983057, 2, 1, 1, 64, 17, 1, 64, "cos"),      # six segments in parts of 32768, the last of 17 documents
]


# (N, Hkv, B, k): rows of the scan's score matrix that eight waves take, at the edges of their range
ROWS_EIGHT = [(2048, 2, 3, 17), (2049, 2, 3, 64), (5000, 4, 2, 1), (8192, 8, 8, 33), (8193, 2, 2, 64), (4100, 8, 33, 20)]


@pytest.mark.parametrize("N,Hkv,B,k", ROWS_EIGHT)
def test_row_selection(N, Hkv, B, k):
    """Scores of float64 to fp32 rounding, and the documents that have them."""
    say(f"row selection N={N} Hkv={Hkv} B={B} k={k}")
    C, d = 8, 64
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6)
    KRb, inv = random_index(53000 + N, N, Hkv, C, d)
    qb, q = S.normal_bf16(53001, (B, 1, Hkv, d))
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    idx, val = msa.msa_score_topk(cfg, dev(qb), dKR, dinv, k)
    torch.cuda.synchronize()
    check_topk_generic(q, KRb, C, N, idx, val, k, "cos", "group", False)


# a scan of four query tiles at the edges between one tile requested ahead of the folding and all (6 or 8 tiles per wave)
FOUR_TILES = [(3072, 8, 2, 8, 64, 32, 1, 16, "cos"), (3073, 8, 1, 8, 64, 32, 1, 16, "dot"), (4096, 8, 1, 8, 128, 24, 1, 9, "cos"),
              (4097, 8, 1, 8, 128, 23, 1, 9, "cos"), (4099, 8, 1, 8, 64, 25, 1, 9, "dot")]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", FOUR_TILES)
def test_scan_of_four_tiles(N, Hkv, r, C, d, B, M, k, sim):
    test_prefill_scoring_k_above_16(N, Hkv, r, C, d, B, M, k, sim)


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", ALL_SCAN)
def test_all_heads_scan(N, Hkv, r, C, d, B, M, k, sim):
    say(f"all-heads scan N={N} Hkv={Hkv} C={C} d={d} B={B} M={M} k={k} {sim}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv * r, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL,
                        sim=msa.MSA_SIM_COS if sim == "cos" else msa.MSA_SIM_DOT)
    KRb, inv = random_index(51000 + N, N, Hkv, C, d)
    qb, q = S.normal_bf16(51001 + N, (B, M, Hkv * r, d))
    KRb[:, 3 * C] = KRb[:, (N - 2) * C]          # two documents with an equal chunk
    inv = 1.0 / np.maximum(np.linalg.norm(KRb, axis=-1), O.EPS_NORM)
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    for pool in (False, True):
        cfg_p = cfg.replace(token_pool=int(pool))
        ws = torch.full((msa.score_topk_workspace_bytes(cfg_p, B, M, k),), 0xFF, dtype=torch.uint8, device="cuda")
        idx, val = msa.msa_score_topk(cfg_p, dev(qb), dKR, dinv if sim == "cos" else None, k, workspace=ws)
        torch.cuda.synchronize()
        check_topk_generic(q, KRb, C, N, idx, val, k, sim, "all", pool, atol=2e-5 if sim == "cos" else 2e-4)


# the same at the edge between queries that the scan's workgroups fold themselves and prepared ones
ALL_FOLDED = [
    (97, 8, 4, 8, 128, 8, 1, 16, "cos"),      # a tile for every wave
    (97, 8, 4, 8, 128, 3, 3, 16, "cos"),      # one query more: prepared
    (33, 4, 8, 16, 64, 16, 1, 5, "cos"),      # two tiles of queries
    (33, 4, 3, 16, 64, 17, 1, 5, "dot"),
    (2100, 2, 1, 1, 128, 6, 5, 9, "dot"),     # four tiles of two heads, the last of 6 queries
    (70, 2, 2, 4, 64, 1, 1, 12, "cos"),       # waves without a tile
    (97, 4, 8, 8, 128, 11, 1, 16, "cos"),     # as many queries as are folded over any index
    (97, 4, 8, 8, 128, 12, 1, 16, "cos"),     # prepared: more of them ...
    (97, 8, 8, 8, 128, 8, 1, 16, "dot"),
    (97, 8, 8, 8, 128, 5, 1, 16, "dot"),      # prepared with eight groups, where four queries are folded
    (97, 8, 8, 8, 128, 4, 1, 16, "dot"),
    (3000, 4, 8, 16, 128, 16, 1, 16, "cos"),  # ... but over an index of 12000 tiles
    (2999, 4, 8, 16, 128, 16, 1, 16, "cos"),
    (70000, 2, 2, 2, 64, 2, 4, 20, "cos"),    # parts of rows
]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", ALL_FOLDED)
def test_all_heads_scan_folds(N, Hkv, r, C, d, B, M, k, sim):
    test_all_heads_scan(N, Hkv, r, C, d, B, M, k, sim)


@pytest.mark.parametrize("pool", [0, 1])
def test_all_heads_scan_lists_in_windows(pool):
    """A bank of 388 parts, of whose lists the buffer holds 380 (32 queries, k = 64): two windows, the second short.
    Against float64 scores on the GPU."""
    N, Hkv, d, B, k = 12700007, 2, 64, 32, 64
    say(f"all-heads scan, lists in windows: N={N} B={B} k={k} pool={pool}")
    cfg = msa.MsaConfig(N, 64, 64, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL, token_pool=pool)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(58000)
    KR, inv = msa.alloc_routing_index(cfg)
    KR.normal_(generator=gen)
    KR[:, -1, :, N % 16:] = 0
    plain = KR.permute(0, 1, 3, 2, 4).reshape(Hkv, -1, d)[:, :N]
    inv.zero_()
    for g in range(Hkv):
        inv[g, :N] = 1.0 / plain[g].float().norm(dim=-1)
    q = torch.randn((B // 4, 4, Hkv, d) if pool else (B, 1, Hkv, d), generator=gen, device="cuda").to(torch.bfloat16)
    ws = torch.full((msa.score_topk_workspace_bytes(cfg, q.shape[0], q.shape[1], k),), 0xFF, dtype=torch.uint8, device="cuda")
    idx, val = msa.msa_score_topk(cfg, q, KR, inv, k, workspace=ws)
    torch.cuda.synchronize()
    x = q.double().reshape(B, Hkv, d)
    x = x / x.norm(dim=-1, keepdim=True)
    for b in range(0, B, 4):                      # four rows of scores at a time
        ref = torch.zeros((4, N), dtype=torch.float64, device="cuda")
        for g in range(Hkv):
            kg = plain[g].double()
            ref += x[b:b + 4, g] @ (kg / kg.norm(dim=-1, keepdim=True)).t().contiguous() / Hkv
        if pool:
            ref = ref.amax(0, keepdim=True)
        for i in range(ref.shape[0]):
            gi, gv = idx.reshape(-1, k)[b // 4 if pool else b + i].long(), val.reshape(-1, k)[b // 4 if pool else b + i].double()
            best = ref[i].topk(k).values
            assert gi.unique().numel() == k and (gv - ref[i][gi]).abs().max() <= 2e-5
            assert (gv - best).abs().max() <= 2e-5    # the k best, in order (up to fp32 rounding of the scores)


# (N, Hkv, r, C, d, B, M, k, sim): the scoring GEMM with more than 16 selected documents
GEMM_K32 = [
    (5003, 2, 2, 8, 128, 1, 300, 32, "cos"),      # one-pass filter, lists shorter than k
    (700, 2, 1, 8, 128, 1, 100, 17, "cos"),       # little work: the scan
    (40, 2, 1, 8, 128, 1, 64, 32, "cos"),
    (3001, 2, 1, 8, 128, 1, 100, 25, "cos"),      # filter, one workgroup of tokens
    (40, 2, 1, 8, 128, 1, 321, 32, "cos"),        # one short split: no filter
    (613, 4, 1, 16, 128, 1, 130, 20, "cos"),      # few tokens, a small bank and no filter: the scan
    (901, 2, 1, 4, 64, 2, 35, 32, "dot"),
    (613, 4, 1, 16, 128, 1, 449, 20, "cos"),      # two-pass form, 32-entry lists
    (301, 2, 1, 4, 64, 2, 161, 32, "dot"),
]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", GEMM_K32)
def test_prefill_scoring_k_above_16(N, Hkv, r, C, d, B, M, k, sim):
    say(f"scoring GEMM N={N} Hkv={Hkv} C={C} d={d} B={B} M={M} k={k} {sim}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv * r, Hkv, d, 1e6, sim=msa.MSA_SIM_COS if sim == "cos" else msa.MSA_SIM_DOT)
    KRb, inv = random_index(53000 + N, N, Hkv, C, d)
    qb, q = S.normal_bf16(53001 + N, (B, M, Hkv * r, d))
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    for pool in (False, True):
        idx, val = msa.msa_score_topk(cfg.replace(token_pool=int(pool)), dev(qb), dKR, dinv if sim == "cos" else None, k)
        torch.cuda.synchronize()
        check_topk_generic(q, KRb, C, N, idx, val, k, sim, "group", pool, atol=2e-5 if sim == "cos" else 2e-4)


# 33 to 63 tokens over a bank that the scan would read twice: the GEMM from 64000 keys a head on (k > 16 or four heads: 320000)
GEMM_TWO_PASSES = [(8000, 8, 1, 8, 128, 33, 1, 8, "cos"), (8001, 8, 2, 8, 128, 3, 21, 16, "cos"), (7999, 8, 1, 8, 128, 40, 1, 8, "cos"),
                   (20003, 8, 1, 8, 128, 35, 1, 24, "cos"), (8200, 8, 1, 8, 128, 32, 1, 8, "cos"), (40001, 4, 1, 8, 128, 63, 1, 5, "cos")]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", GEMM_TWO_PASSES)
def test_scoring_gemm_of_two_passes(N, Hkv, r, C, d, B, M, k, sim):
    test_prefill_scoring_k_above_16(N, Hkv, r, C, d, B, M, k, sim)


# score-matrix scans at the edge between plain and streaming loads of the index (128 MB; a scan per group in two passes: 300 MB),
# tails of half a tile
STREAMED = [(7812, 8, 1, 8, 128, 1, 1, 9, "cos"), (7813, 8, 1, 8, 128, 9, 1, 9, "cos"), (7815, 8, 1, 8, 128, 2, 1, 16, "dot"),
            (7813, 8, 2, 8, 128, 20, 1, 16, "cos"), (31253, 4, 1, 8, 64, 3, 1, 8, "cos"), (18311, 8, 1, 8, 128, 2, 1, 9, "cos"),
            (18310, 8, 1, 8, 128, 33, 1, 9, "dot"), (18311, 8, 1, 8, 128, 33, 1, 9, "dot")]


@pytest.mark.parametrize("scope", ["group", "all"])
@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", STREAMED)
def test_scans_with_streaming_loads(N, Hkv, r, C, d, B, M, k, sim, scope):
    (test_all_heads_scan if scope == "all" else test_prefill_scoring_k_above_16)(N, Hkv, r, C, d, B, M, k, sim)


# all heads over 128 MB of documents of one and two chunks: streaming loads up to eight queries, plain ones for more; four chunks
@pytest.mark.parametrize("N,C,B", [(62501, 1, 8), (62501, 1, 9), (31253, 2, 17), (15627, 4, 9)])
def test_all_heads_scan_loads_of_short_documents(N, C, B):
    test_all_heads_scan(N, 8, 1, C, 128, B, 1, 9, "cos")


@pytest.mark.parametrize("M", [250, 700, 2000])
def test_token_pooling_of_many_documents(M):
    """One query head: the tokens' scores are alike and most of their listed documents reach the floor: 1300 and about
    3000 of them (ranked from the table in LDS), and 6422 (more than it takes: rounds over the lists)."""
    test_prefill_scoring_k_above_16(9001, 1, 1, 4, 64, 1, M, 16, "cos")


@pytest.mark.parametrize("M", [70, 330])
def test_prefill_scoring_k_above_16_neighbouring_winners(M):
    """The best documents of every token lie side by side: more of them in one list of the one-pass filter than it
    holds, so every token block is redone by the two-pass form with 32-entry lists (M = 70: the scan's case)."""
    N, Hkv, C, d, k = 4000, 2, 8, 128, 24
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6)
    KRb, _ = random_index(54000, N, Hkv, C, d)
    qb, q = S.normal_bf16(54001, (1, M, Hkv, d))
    qb, q = qb & 0x7FFF, np.abs(q)                # every query component positive ...
    docs = KRb.reshape(Hkv, N, C, d)
    docs[:, 1000:1100] = np.abs(docs[:, 1000:1100])   # ... and so are the keys of a hundred neighbours
    inv = 1.0 / np.maximum(np.linalg.norm(KRb, axis=-1), O.EPS_NORM)
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    idx, val = msa.msa_score_topk(cfg, dev(qb), dKR, dinv, k)
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    assert got.min() >= 1000 and got.max() < 1100
    check_topk_generic(q, KRb, C, N, idx, val, k, "cos", "group", False)


# (N, Hkv, r, C, d, B, M, k, sim): more tokens than a pass of the scan -> the wide kernel and its selection
ALL_WIDE = [
    (70, 8, 1, 8, 128, 1, 33, 17, "cos"),         # one token more than the scan takes, a ragged unit
    (5003, 8, 2, 8, 128, 2, 75, 32, "cos"),       # three token blocks, the last ragged
    (1037, 4, 2, 16, 128, 1, 65, 64, "cos"),      # one document per tile, the largest k
    (4099, 8, 1, 1, 64, 1, 70, 20, "dot"),        # hi and lo rows, sixteen documents per tile
    (30011, 2, 1, 2, 64, 1, 300, 9, "cos"),       # two segments of the bank
    (333, 2, 1, 4, 128, 1, 1030, 3, "cos"),       # two passes of tokens
    (5, 2, 1, 8, 64, 3, 20, 5, "dot"),            # as many documents as are selected
    (70001, 2, 1, 2, 64, 1, 35, 20, "cos"),       # one segment longer than a selecting workgroup's registers
    (33001, 2, 1, 8, 128, 1, 35, 64, "cos"),      # ... and with the one-pass filter
]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", ALL_WIDE)
def test_all_heads_wide(N, Hkv, r, C, d, B, M, k, sim):
    test_all_heads_scan(N, Hkv, r, C, d, B, M, k, sim)


# the same at the edges of the kernel that reads a key once for 65 to 160 rows: numbers of row tiles, units that end inside a
# wave's keys, from 64 documents on
ALL_ROWS = [(37, 8, 1, 8, 128, 1, 64, 9, "cos"), (37, 8, 1, 8, 128, 1, 65, 9, "cos"), (1003, 8, 2, 8, 128, 1, 96, 16, "cos"),
            (2051, 8, 4, 8, 128, 1, 97, 32, "cos"), (5, 8, 1, 8, 128, 2, 64, 5, "cos"), (520, 8, 4, 8, 128, 3, 53, 12, "cos"),
            (999, 8, 1, 8, 128, 1, 129, 16, "cos"), (4100, 8, 2, 8, 128, 1, 160, 8, "cos"), (300, 8, 1, 8, 128, 1, 161, 8, "cos"),
            # ten tiles of rows with a round of units less than blocks of 64 rows take, eight in one round, and just not
            (5440, 8, 1, 8, 128, 1, 130, 8, "cos"), (5441, 8, 1, 8, 128, 1, 129, 16, "cos"), (8192, 8, 1, 8, 128, 1, 160, 8, "cos"),
            (8193, 8, 1, 8, 128, 1, 145, 8, "cos"), (8192, 8, 1, 8, 128, 1, 128, 8, "cos"), (8193, 8, 1, 8, 128, 1, 97, 8, "cos"),
            (10881, 8, 1, 8, 128, 1, 131, 8, "cos"), (20001, 8, 1, 8, 128, 1, 100, 8, "cos")]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", ALL_ROWS)
def test_all_heads_wide_rows(N, Hkv, r, C, d, B, M, k, sim):
    test_all_heads_scan(N, Hkv, r, C, d, B, M, k, sim)


# the same with streaming loads of the index: pooled from 128 MB on, else from 300 MB on with one block of tokens
@pytest.mark.parametrize("N,M", [(7813, 40), (7813, 70), (7815, 100), (7814, 131), (7812, 150), (16384, 33), (16387, 64), (18311, 33),
                                 (18313, 64), (18312, 90)])
def test_all_heads_wide_rows_with_streaming_loads(N, M):
    test_all_heads_scan(N, 8, 1, 8, 128, 1, M, 9, "cos")


# tokens pooled by document: one token more than the scan takes, several blocks of tokens, batch rows, parts of one document
POOL_DOCS = [(700, 2, 2, 8, 128, 1, 33, 20, "cos"), (1030, 4, 1, 8, 128, 2, 100, 9, "cos"), (64, 4, 2, 8, 128, 1, 330, 64, "cos"),
             (515, 2, 1, 8, 128, 1, 1000, 5, "cos"), (2600, 8, 1, 8, 128, 4, 66, 33, "cos"), (40, 8, 1, 8, 128, 1, 40, 40, "cos"),
             (5, 2, 1, 8, 128, 1, 49, 1, "cos")]


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", POOL_DOCS)
def test_token_pooling_by_document(N, Hkv, r, C, d, B, M, k, sim):
    test_all_heads_scan(N, Hkv, r, C, d, B, M, k, sim)


# the edges of the rule: the fewest documents that are pooled by document
POOL_DOCS_LEAST = [(9, 8, 1, 8, 128, 1, 64, 9, "cos"), (64, 8, 1, 8, 128, 1, 150, 16, "cos"), (1999, 8, 1, 8, 128, 1, 130, 3, "cos")]
# ... and just not: too few documents, more blocks than those of 64 tokens, a token too many
POOL_TOKENS = [(8, 8, 1, 8, 128, 1, 64, 8, "cos"), (62, 8, 1, 8, 128, 1, 150, 16, "cos"), (1998, 8, 1, 8, 128, 1, 130, 3, "cos"),
               (300, 4, 1, 8, 128, 3, 40, 5, "cos"), (300, 2, 1, 8, 128, 1, 1025, 4, "cos")]


def pooled_by_document(N, Hkv, B, M, k):
    """Whether the tokens of an all-heads call (cosine, d = 128, C = 8) are pooled by document: few enough blocks of tokens, enough
    documents, and buffers that fit where those of a selection per token lie."""
    d, up = 128, lambda b: (b + 255) // 256 * 256
    blocks, tiles = (M + 159) // 160, (N + 1) // 2
    if M <= 32 or B * M > 1024 or B * blocks > (B * M + 63) // 64:
        return False
    if tiles < (32 if blocks == 1 and M > 96 else 5) or (128 < M <= 160 and k < 16 and tiles < 1000):
        return False
    seg = -(-N // -(-N // max(64, 5 * 2**20 // (B * M))))
    common = up(B * M * Hkv * d * 4) + up(B * M * Hkv * 4)
    per_token = up(Hkv * -(-B * M // 64) * 4 * d * 32) + up(B * M * k * 8) + up(B * M * min(N, (seg + 63) // 64 * 64) * 4)
    by_doc = (up(Hkv * B * -(-M // 16) * d * 32) + up(B * blocks * N * 4) + up(B * 512 * 4) + 2 * up(B * 4) + up(B * N * 4) +
              up(B * N * 8))
    assert msa.score_topk_workspace_bytes(msa.MsaConfig(N, 64, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL, token_pool=1),
                                          B, M, k) >= common + per_token
    return by_doc <= per_token


@pytest.mark.parametrize("N,Hkv,r,C,d,B,M,k,sim", POOL_DOCS_LEAST + POOL_TOKENS)
def test_token_pooling_at_the_edges_of_its_rule(N, Hkv, r, C, d, B, M, k, sim):
    assert all(pooled_by_document(n, h, b, m, kk) == (n > 5) for n, h, _, _, _, b, m, kk, _ in POOL_DOCS)
    assert pooled_by_document(N, Hkv, B, M, k) == ((N, Hkv, r, C, d, B, M, k, sim) in POOL_DOCS_LEAST)
    test_all_heads_scan(N, Hkv, r, C, d, B, M, k, sim)


@pytest.mark.parametrize("N,copies,k,zeros", [(6000, 3000, 16, 0), (3000, 100, 64, 39), (9000, 0, 64, 40)])
def test_token_pooling_of_copies_and_zeros(N, copies, k, zeros):
    """The best documents are copies of one (more of them than the last kernel's LDS takes), zeros of the 40 tokens are
    zeros: copies are selected in their order, and with zeros alone the first k documents.  Against float64 scores."""
    Hkv, d, M = 4, 128, 40
    say(f"token pooling N={N} copies={copies} k={k} zeros={zeros}")
    cfg = msa.MsaConfig(N, 64, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL, token_pool=1)
    KRb, _ = random_index(59000 + N, N, Hkv, 8, d)
    qb, q = S.normal_bf16(59001, (1, M, Hkv, d))
    qb, q = qb.copy(), q.copy()
    qb[:, M - zeros:], q[:, M - zeros:] = 0, 0
    at = np.arange(N - 1, N - 1 - copies, -1)
    if copies:
        KRb.reshape(Hkv, N, 8, d)[:, at, :] = q[0, 0][:, None, None, :]   # what the first token asks for, in every chunk
    inv = 1.0 / np.maximum(np.linalg.norm(KRb, axis=-1), O.EPS_NORM)
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    ws = torch.full((msa.score_topk_workspace_bytes(cfg, 1, M, k),), 0xFF, dtype=torch.uint8, device="cuda")
    idx, val = msa.msa_score_topk(cfg, dev(qb), dKR, dinv, k, workspace=ws)
    torch.cuda.synchronize()
    _, ov, s = O.score_topk(q, KRb, 8, k, select_scope="all", token_pool=True)
    gi, gv = idx.cpu().numpy().reshape(-1), val.cpu().numpy().reshape(-1)
    assert len(set(gi.tolist())) == k
    assert np.max(np.abs(gv - np.asarray(s, dtype=np.float64).reshape(-1)[gi])) <= 2e-5
    assert np.max(np.abs(gv - np.asarray(ov).reshape(-1))) <= 2e-5
    if copies:
        n = min(copies, k)
        assert np.array_equal(gi[:n], np.arange(N - copies, N - copies + n))
    elif zeros == M:
        assert np.array_equal(gi, np.arange(k)) and np.all(gv == 0)


def test_token_pooling_of_nothing_but_zeros():
    """A question of zeros takes no longer than another one: of the documents that tie the first k go on, not k of every
    workgroup (which took 1.7 times as long).  A question that is not a number selects nothing."""
    N, Hkv, C, d, M, k = 8192, 8, 8, 128, 150, 32
    say("token pooling of a question of zeros")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL, token_pool=1)
    keys, KR = device_index(61001, Hkv, N * C, d)
    inv = 1.0 / keys.float().norm(dim=-1)
    q = torch.randn((1, M, Hkv, d), generator=torch.Generator("cuda").manual_seed(1), device="cuda").to(torch.bfloat16)
    _, _, plain = call_us(cfg, q, KR, inv, k)
    idx, val, zeros = call_us(cfg, torch.zeros_like(q), KR, inv, k)
    assert torch.equal(idx.view(-1), torch.arange(k, dtype=torch.int32, device="cuda")) and bool((val == 0).all())
    say(f"  {plain:.0f} us, zeros {zeros:.0f}")
    assert zeros <= 1.3 * plain
    idx, val, _ = call_us(cfg, torch.full_like(q, float("nan")), KR, inv, k)
    assert bool((idx == -1).all()) and bool((val == float("-inf")).all())


@pytest.mark.parametrize("N,k,M", [(40, 40, 64), (9001, 20, 40), (600, 64, 330)])
def test_token_pooling_of_what_is_not_a_number(N, k, M):
    """Pooled by document as from a selection per token: a question that holds an infinity in every token lists the first k
    documents without a score, such tokens beside others change nothing, and neither does a document without a score, which
    goes on the list only where there are no others."""
    Hkv, C, d = 8, 8, 128
    say(f"token pooling of what is not a number N={N} k={k} M={M}")
    assert pooled_by_document(N, Hkv, 1, M, k)
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL, token_pool=1)
    keys, KR = device_index(62001, Hkv, N * C, d)
    inv = torch.ones((Hkv, KR.shape[1] * 16), device="cuda")
    inv[:, :N * C] = 1.0 / keys.float().norm(dim=-1)
    q = torch.randn((1, M, Hkv, d), generator=torch.Generator("cuda").manual_seed(2), device="cuda").to(torch.bfloat16)
    bad = q.clone()
    bad[:, :, 3, 5] = float("inf")
    idx, val = msa.msa_score_topk(cfg, bad, KR, inv, k)
    assert torch.equal(idx.view(-1), torch.arange(k, dtype=torch.int32, device="cuda")) and bool(val.isnan().all())
    idx, val = msa.msa_score_topk(cfg, q, KR, inv, k)
    for what in (float("inf"), float("nan")):
        one = q.clone()
        one[0, 1:, 3, 5] = what
        first = msa.msa_score_topk(cfg, one, KR, inv, k)
        alone = q.clone()
        alone[0, 1:] = q[0, :1]
        second = msa.msa_score_topk(cfg, alone, KR, inv, k)
        assert torch.equal(first[0], second[0]) and torch.equal(first[1], second[1])
    doc = int(idx[0, 0, 0, 0])                        # the best document
    inv[:, doc * C:doc * C + C] = float("nan")
    idx2, val2 = msa.msa_score_topk(cfg, q, KR, inv, k)
    scored = ~val2.isnan()
    assert int(scored.sum()) == (k - 1 if k == N else k) and (k < N or int(idx2[~scored]) == doc)
    assert torch.equal(idx2[scored][:k - 1], idx.view(-1)[1:]) and torch.equal(val2[scored][:k - 1], val.view(-1)[1:])


# (N, Hkv, C, d, B, M, k, scope, pool): a row's k best where every document ties
ALL_TIED = [
    (97656, 8, 8, 128, 8, 1, 32, "group", 0),     # candidate lists of long streams and their merge
    (40001, 8, 8, 128, 3, 1, 8, "group", 0),
    (9000, 2, 8, 64, 3, 1, 16, "group", 0),       # row top-k, four waves, part of the row beyond the registers
    (30001, 2, 1, 64, 2, 1, 64, "all", 0),        # sixteen waves
    (40007, 2, 1, 64, 2, 1, 33, "all", 0),        # rows in parts, the last of 7239 documents
    (70001, 2, 1, 64, 1, 40, 33, "all", 0),       # wide kernel, scores of hi and lo parts
    (9001, 8, 8, 128, 1, 50, 20, "all", 0),       # ... and behind the one-pass filter
    (30011, 2, 8, 128, 1, 400, 9, "all", 1),      # pooled by document
    (30011, 2, 8, 128, 1, 1100, 9, "all", 1),     # two passes of tokens, a selection per token in segments, pooled from those
    (30011, 4, 8, 128, 3, 40, 9, "all", 1),       # blocks of tokens more than the rows: the same in one pass
]


@pytest.mark.parametrize("N,Hkv,C,d,B,M,k,scope,pool", ALL_TIED)
def test_queries_of_zeros(N, Hkv, C, d, B, M, k, scope, pool):
    """Empty slots of a batch and padding of a question: a query of zeros scores zero with every document, so its
    selection is the first k; the queries beside it are what they are without it."""
    say(f"queries of zeros N={N} Hkv={Hkv} C={C} d={d} B={B} M={M} k={k} {scope} pool={pool}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, token_pool=pool,
                        select_scope=msa.MSA_SCOPE_ALL if scope == "all" else msa.MSA_SCOPE_GROUP)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(60000 + N)
    KR, inv = msa.alloc_routing_index(cfg)
    KR.normal_(generator=gen)
    inv.copy_(KR.float().pow(2).sum((2, 4)).rsqrt().reshape(Hkv, -1))
    q = torch.randn((B, M, Hkv, d), generator=gen, device="cuda").to(torch.bfloat16)
    flat = q.view(B * M, Hkv, d)
    zero = torch.arange(B * M, device="cuda") % 2 == 1 if not pool else torch.ones(B * M, dtype=torch.bool, device="cuda")
    if B * M == 2:
        zero[1] = True
    flat[zero] = 0
    idx, val = msa.msa_score_topk(cfg, q, KR, inv, k)
    torch.cuda.synchronize()
    S_ = 1 if scope == "all" else Hkv
    first = torch.arange(k, dtype=torch.int32, device="cuda")
    if pool:
        assert torch.equal(idx, first.expand_as(idx)) and bool((val == 0).all())
        return
    idx, val = idx.reshape(B * M, S_, k), val.reshape(B * M, S_, k)
    assert torch.equal(idx[zero], first.expand_as(idx[zero])) and bool((val[zero] == 0).all())
    rest = flat[~zero].clone().view(1, -1, Hkv, d)
    if rest.shape[1] == B * M:
        return
    alone, score = msa.msa_score_topk(cfg, rest, KR, inv, k)
    torch.cuda.synchronize()
    # (fewer queries may take another kernel: the same documents but for ties of the rounded scores)
    assert (val[~zero] - score.reshape(-1, S_, k)).abs().max() <= 2e-5
    assert (idx[~zero] != alone.reshape(-1, S_, k)).float().mean() <= 0.01


@pytest.mark.parametrize("k", [8, 32])
@pytest.mark.parametrize("what", ["zeros", "copies"])
def test_merge_of_tied_lists(what, k):
    """Long streams whose lists hold documents that tie: the first k of them, in about the time of a call without ties (the
    merge took the call to 1.5 to 1.9 times that where every entry of every list went on to be ranked)."""
    N, Hkv, C, d, B = 97656, 8, 8, 128, 8
    say(f"merge of lists that tie: {what} k={k}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6)
    keys, KR = device_index(61000, Hkv, N * C, d)
    q = torch.randn((B, 1, Hkv, d), generator=torch.Generator("cuda").manual_seed(k), device="cuda").to(torch.bfloat16)
    inv = torch.zeros((Hkv, cfg.n_tiles * 16), device="cuda")
    inv[:, :N * C] = 1.0 / keys.float().norm(dim=-1)
    _, _, plain = call_us(cfg, q, KR, inv, k)
    at = torch.arange(k, device="cuda")
    if what == "zeros":
        q[-2:] = 0
    else:   # what the first query asks for, in every chunk of 3000 documents
        at = torch.randperm(N, generator=torch.Generator("cuda").manual_seed(7), device="cuda")[:3000].sort().values
        keys = keys.clone().view(Hkv, N, C, d)
        keys[:, at] = q[0, 0][:, None, None, :]
        KR = keys.reshape(Hkv, -1, 16, d // 8, 8).transpose(2, 3).contiguous()
        inv[:, :N * C] = 1.0 / keys.float().norm(dim=-1).reshape(Hkv, -1)
    idx, val, tied = call_us(cfg, q, KR, inv, k)
    idx, val = idx[:, 0], val[:, 0]
    rows = idx[-2:] if what == "zeros" else idx[:1]
    assert torch.equal(rows, at[:k].int().expand_as(rows))
    assert bool((val[-2:] == 0).all()) if what == "zeros" else (val[0] - 1).abs().max() <= 2e-5
    say(f"  {plain:.0f} us, with ties {tied:.0f}")
    assert tied <= 1.35 * plain


@pytest.mark.parametrize("C,d", [(8, 64), (4, 128)])
def test_all_heads_wide_takes_any_norms(C, d):
    """An index whose reciprocal norms are not those of its keys (a hundred times them, more or less): scored as it is
    wherever the one-pass filter, whose error band is that of unit keys, is not announced."""
    N, Hkv, M, k = 3000, 2, 40, 8
    say(f"all-heads scoring with norms of its own C={C} d={d}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL)
    KRb, inv = random_index(59000 + d, N, Hkv, C, d)
    inv = (inv * np.random.default_rng(59001).uniform(50, 150, inv.shape)).astype(np.float32).astype(np.float64)
    qb, q = S.normal_bf16(59002, (1, M, Hkv, d))
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    idx, val = msa.msa_score_topk(cfg, dev(qb), dKR, dinv, k)
    torch.cuda.synchronize()
    x = q[0] / np.linalg.norm(q[0], axis=-1, keepdims=True)                     # [M][Hkv][d]
    s = sum((x[:, g] @ KRb[g].T) * inv[g] for g in range(Hkv)) / Hkv
    s = s.reshape(M, N, C).max(-1)
    want = np.sort(s, axis=-1)[:, ::-1][:, :k]
    got = idx.cpu().numpy()[0, :, 0]
    # scores of up to ~60 with queries carried to 16 bits and fp32 sums: 2e-5 of the largest at most
    assert np.abs(np.take_along_axis(s, got.astype(np.int64), -1) - want).max() <= 2e-5 * want.max()
    assert np.abs(val.cpu().numpy()[0, :, 0] - want).max() <= 2e-5 * want.max()


# 33 to 63 tokens above the lines of the GEMM that stands in for two passes of the scan, and below (24 of 20000)
@pytest.mark.parametrize("N,Hkv,k", [(16000, 8, 8), (16001, 8, 12), (20000, 8, 24), (40003, 8, 24), (40001, 4, 8)])
def test_scoring_of_two_passes_takes_any_norms(N, Hkv, k):
    """As test_all_heads_wide_takes_any_norms, a selection per KV group."""
    C, d, B = 8, 128, 40
    say(f"scoring of two passes with norms of its own N={N} Hkv={Hkv} k={k}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6)
    keys, KR = device_index(60000 + N, Hkv, N * C, d)
    inv = torch.zeros((Hkv, cfg.n_tiles * 16), device="cuda")
    inv[:, :N * C] = 1.0 / keys.float().norm(dim=-1)
    inv *= 50 + 100 * torch.rand(inv.shape, generator=torch.Generator("cuda").manual_seed(k), device="cuda")
    q = dev(S.normal_bf16(60001, (B, 1, Hkv, d))[0])
    idx, val = msa.msa_score_topk(cfg, q, KR, inv, k)
    torch.cuda.synchronize()
    x = q[:, 0].double()
    x = x / x.norm(dim=-1, keepdim=True)
    for g in range(Hkv):
        s = ((x[:, g] @ keys[g].double().T.contiguous()) * inv[g, :N * C].double()).reshape(B, N, C).amax(-1)
        want = s.topk(k, dim=1).values
        # (the bound of test_all_heads_wide_takes_any_norms)
        assert (s.gather(1, idx[:, 0, g].long()) - want).abs().max() <= 2e-5 * want.max()
        assert (val[:, 0, g].double() - want).abs().max() <= 2e-5 * want.max()


@pytest.mark.parametrize("pool", [0, 1])
@pytest.mark.parametrize("k", [8, 16])
def test_scoring_of_two_passes_of_not_a_number(k, pool):
    """Queries that are not numbers select what they select in a call of one pass; the others are as they are alone."""
    N, Hkv, C, d, B = 8100, 8, 8, 128, 20
    say(f"scoring of two passes, queries that are not numbers k={k} pool={pool}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, token_pool=pool)
    keys, KR = device_index(60700, Hkv, N * C, d)
    inv = torch.zeros((Hkv, cfg.n_tiles * 16), device="cuda")
    inv[:, :N * C] = 1.0 / keys.float().norm(dim=-1)
    q = dev(S.normal_bf16(60701, (B, 2, Hkv, d))[0])
    q[3], q[5, 1, 2], q[16, 0], q[19, 1, :, 7] = (float(x) for x in ("nan", "nan", "-nan", "inf"))
    idx, val = msa.msa_score_topk(cfg, q, KR, inv, k)
    parts = [msa.msa_score_topk(cfg, q[b:b + 10].contiguous(), KR, inv, k) for b in (0, 10)]
    torch.cuda.synchronize()
    one_i, one_v = (torch.cat([p[i] for p in parts]) for i in range(2))
    nan = torch.isnan(one_v)
    assert bool(nan[3].all()) and torch.equal(torch.isnan(val), nan) and torch.equal(idx[nan], one_i[nan])
    assert torch.equal(torch.signbit(val[nan]), torch.signbit(one_v[nan]))
    # both carry the queries as hi and lo parts: scores to fp32 rounding, other documents only where they tie to that
    assert (val[~nan] - one_v[~nan]).abs().max() <= 2e-6
    assert (idx != one_i).float().mean() <= 0.01


@pytest.mark.parametrize("copies,d", [(300, 64), (4000, 64), (300, 128), (4000, 128)])
def test_all_heads_wide_more_candidates_than_k(copies, d):
    """Copies of one document tie exactly: all of them are candidates of every token (4000: more than the selection
    keeps on chip, so the row goes through it in windows); ties go to the lower index."""
    N, Hkv, C, M, k = 6000, 2, 8, 40, 12
    say(f"all-heads selection with {copies} copies of the best document, d={d}")
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL)
    KRb, _ = random_index(52000, N, Hkv, C, d)
    qb, q = S.normal_bf16(52001, (1, M, Hkv, d))
    rng = np.random.default_rng(52002)
    at = rng.permutation(N)[:copies]
    first = KRb.reshape(Hkv, N, C, d)
    first[:, at] = np.abs(first[:, at[:1]])
    qb = qb & 0x7FFF                              # every query component positive: the copies are every token's best
    q = np.abs(q)
    inv = 1.0 / np.maximum(np.linalg.norm(KRb, axis=-1), O.EPS_NORM)
    dKR, dinv = upload_oracle_index(cfg, KRb, inv)
    idx, val = msa.msa_score_topk(cfg, dev(qb), dKR, dinv, k)
    torch.cuda.synchronize()
    want = np.sort(at)[:k]
    assert np.array_equal(idx.cpu().numpy(), np.broadcast_to(want, (1, M, 1, k)))
    _, s = O.score_topk(q, KRb, C, k, "cos", "all", False)[1:]
    assert np.allclose(val.cpu().numpy(), s[..., want], rtol=0, atol=2e-5)


# (N, Hkv, M, k, copies, zeros): several segments, d = 128 and eight chunks: candidates wait for the last segment
ALL_LISTED = [
    (20000, 2, 1000, 32, 0, 0),       # four segments
    (20011, 4, 700, 64, 0, 3),        # a query of zeros in three: exact from its first segment on
    (20000, 2, 600, 12, 300, 0),      # more candidates than wait: exact winners from the segment on where they do not fit
    (9000, 2, 1024, 9, 5000, 5),      # more than the selection holds
    (5300, 8, 1000, 64, 100, 0),      # two segments
]


@pytest.mark.parametrize("N,Hkv,M,k,copies,zeros", ALL_LISTED)
def test_all_heads_wide_candidates_of_all_segments(N, Hkv, M, k, copies, zeros):
    """The same winners and the same exact scores, bit for bit, as where every segment's candidates are scored at once,
    which a workspace without room for the lists does; and the scores of float64."""
    say(f"all-heads lists N={N} Hkv={Hkv} M={M} k={k} copies={copies} zeros={zeros}")
    C, d = 8, 128
    cfg = msa.MsaConfig(N, 8 * C, 8, Hkv, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(61000 + N + k)
    KR, inv = msa.alloc_routing_index(cfg)
    KR.normal_(generator=gen)
    q = torch.randn((1, M, Hkv, d), generator=gen, device="cuda").to(torch.bfloat16)
    if copies:  # [Hkv][tiles][d/8][16][8], two documents per tile
        q = q.abs()
        docs = KR.view(Hkv, -1, d // 8, 2, 8, 8)
        at = torch.randperm(N, generator=gen, device="cuda")[:copies]
        docs[:, at // 2, :, at % 2] = docs[:, 0, :, 0].abs().unsqueeze(0)
    if zeros:
        q[:, ::zeros] = 0
    inv.copy_(KR.float().pow(2).sum((2, 4)).rsqrt().reshape(Hkv, -1))
    size = msa.score_topk_workspace_bytes(cfg, 1, M, k)
    least = size - (M * 160 * 8 + 255) // 256 * 256 - (M * 8 + 255) // 256 * 256
    got = []
    for n in (size, least):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        got.append(msa.msa_score_topk(cfg, q, KR, inv, k, workspace=ws))
        torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    idx, val = got[0][0][0, :, 0].long(), got[0][1][0, :, 0]
    x = q[0].double()
    x = x / x.norm(dim=-1, keepdim=True).clamp_min(1e-12)
    keys = msa.untile_routing_keys(cfg, KR).double().reshape(Hkv, N, C, d)
    s = None
    for g in range(Hkv):
        kg = keys[g] / keys[g].norm(dim=-1, keepdim=True)
        part = x[:, g] @ kg.reshape(N * C, d).t()
        s = part if s is None else s.add_(part)
    s = (s / Hkv).reshape(M, N, C).amax(-1)
    assert (s.topk(k, dim=1).values - val.double()).abs().max() <= 2e-5
    assert (s.gather(1, idx) - val.double()).abs().max() <= 2e-5


@pytest.mark.parametrize("N,Hkv,G,P,d,first,count", [(5, 3, 56, 8, 64, 1, 3), (3, 1, 24, 24, 128, 0, 3), (7, 5, 256, 64, 128, 6, 1),
                                                        (5, 2, 512, 128, 64, 1, 4)])
def test_pool_chunks_by_pairs(N, Hkv, G, P, d, first, count):
    """Pooled bank where the (document, head) pairs do not fill the workgroups, chunks do not fill a batch of loads, and
    a part of the bank is addressed; a bf16 mean is the rounded exact one, or its neighbour where the exact mean lies
    within fp32 summation error (P terms of at most ~6, rotation angles to ~1e-6) of a rounding tie."""
    cfg = msa.MsaConfig(N, G, P, Hkv, Hkv, d, 1e4)
    Kb, K = S.normal_bf16(55000, (N, Hkv, G, d))
    Vb, V = S.normal_bf16(55001, (N, Hkv, G, d))
    lens = np.maximum(1, (np.arange(N) * 37 + 5) % (G + 1)).astype(np.int32)
    for ragged in (False, True):
        c = cfg.replace(doc_lens=torch.from_numpy(lens).cuda() if ragged else None)
        Kbar = torch.full((N, Hkv, G // P, d), 7.0, dtype=torch.bfloat16, device="cuda")
        Vbar = Kbar.clone()
        kw = dict(pooled_lens=torch.zeros(N, dtype=torch.int32, device="cuda")) if ragged else {}
        msa.msa_pool_kv(c, dev(Kb), dev(Vb), doc_begin=first, doc_count=count, Kbar=Kbar, Vbar=Vbar, **kw)
        torch.cuda.synchronize()
        for X, got in ((O.rope(K, np.arange(G), 1e4), Kbar), (V, Vbar)):
            got = got.float().cpu().numpy().astype(np.float64)
            assert np.all(got[:first] == 7.0) and np.all(got[first + count:] == 7.0)
            for i in range(first, first + count):
                n = int(lens[i]) if ragged else G
                for j in range(G // P):
                    rows = X[i, :, j * P:min(n, (j + 1) * P)]
                    want = rows.mean(1) if rows.shape[1] else np.zeros((Hkv, d))
                    assert np.abs(got[i, :, j] - want).max() <= 2.0 ** -8 * np.abs(want).max() + 1e-5


@pytest.mark.parametrize("G,P,d", [(256, 128, 64), (64, 32, 64), (128, 32, 128), (512, 256, 128)])
def test_routing_keys_by_batches(G, P, d):
    """Chunks of four and eight loads (one batch of eight), of sixteen and of sixty-four (batches of sixteen): a key is the
    rounded exact mean, or its neighbour at a tie, as for the pooled bank above."""
    N, Hkv = 5, 2
    Kb, K = S.normal_bf16(57000, (N, Hkv, G, d))
    lens = (np.arange(N) * 53 % G + 1).astype(np.int32)
    for ragged in (False, True):
        cfg = msa.MsaConfig(N, G, P, Hkv, Hkv, d, 1e4, doc_lens=torch.from_numpy(lens).cuda() if ragged else None)
        KR, inv = msa.msa_build_routing_keys(cfg, dev(Kb))
        torch.cuda.synchronize()
        got = msa.untile_routing_keys(cfg, KR).float().cpu().numpy().astype(np.float64).reshape(Hkv, N, G // P, d)
        for i in range(N):
            n = int(lens[i]) if ragged else G
            for j in range(G // P):
                first = j * P if j * P < n else 0
                want = K[i, :, first:min(n, first + P)].mean(1)
                assert np.abs(got[:, i, j] - want).max() <= 2.0 ** -8 * np.abs(want).max() + 1e-5


@pytest.mark.parametrize("G,P,d,first,count", [(64, 8, 64, 0, 5), (512, 64, 128, 1, 3), (256, 16, 128, 2, 3), (1024, 64, 64, 4, 1)])
def test_routing_keys_by_runs(G, P, d, first, count):
    """Eight and sixteen chunks per document, none short: eight keys leave together.  Keys as above, the norms those of the
    rounded keys (fp32 sums and a square root: 2e-6 of the value), and no slot of a document that was not asked for."""
    N, Hkv, C = 5, 3, G // P
    Kb, K = S.normal_bf16(57100, (N, Hkv, G, d))
    cfg = msa.MsaConfig(N, G, P, Hkv, Hkv, d, 1e4)
    KR, inv = msa.alloc_routing_index(cfg)
    KR.fill_(7.0)
    inv.fill_(7.0)
    msa.msa_build_routing_keys(cfg, dev(Kb), doc_begin=first, doc_count=count, KR=KR, inv_norm=inv)
    torch.cuda.synchronize()
    got = msa.untile_routing_keys(cfg, KR).float().cpu().numpy().astype(np.float64).reshape(Hkv, N, C, d)
    norm = inv.cpu().numpy().astype(np.float64).reshape(Hkv, -1)[:, :N * C].reshape(Hkv, N, C)
    there = np.arange(N)[(np.arange(N) >= first) & (np.arange(N) < first + count)]
    rest = np.setdiff1d(np.arange(N), there)
    want = K.reshape(N, Hkv, C, P, d).mean(3).transpose(1, 0, 2, 3)
    assert np.abs(got[:, there] - want[:, there]).max() <= 2.0 ** -8 * np.abs(want).max() + 1e-5
    assert np.abs(norm[:, there] * np.linalg.norm(got[:, there], axis=-1) - 1).max() <= 2e-6
    assert np.all(got[:, rest] == 7.0) and np.all(norm[:, rest] == 7.0)


@pytest.mark.parametrize("d", [128, 64])
def test_chunk_of_more_elements_than_an_int_counts(d):
    """One document in one chunk of 2^31 elements and 4096 rows more, zero but for rows on both sides of the 2^31st
    element: sums of integers, exact in fp32, and the mean rounded once (2^-8 of it).  The pooled keys likewise in the pairs
    whose angle stays under 1e-5 over the whole chunk."""
    half = 2 ** 31 // d
    G = half + 4096
    say(f"chunk of {G} rows of {d}")
    cfg = msa.MsaConfig(1, G, G, 1, 1, d, 1e38)
    X = torch.zeros((1, 1, G, d), dtype=torch.bfloat16, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(57200)
    for at, n in ((0, 40), (half - 24, 64), (G - 200, 200)):
        X[0, 0, at:at + n] = torch.randint(1, 9, (n, d), generator=gen, device="cuda").to(torch.bfloat16)
    want = sum(X[0, 0, i:i + (1 << 22)].float().sum(0).double() for i in range(0, G, 1 << 22)) / G
    KR, inv = msa.msa_build_routing_keys(cfg, X)
    Kbar, Vbar = msa.msa_pool_kv(cfg, X, X)
    torch.cuda.synchronize()
    still = [u for u in range(d) if 1e38 ** (-2.0 * (u % (d // 2)) / d) * G < 1e-5]
    assert len(still) >= d // 2
    assert ((Kbar.reshape(d).double() - want).abs() <= (2.0 ** -8 + 2e-5) * want)[still].all()
    key = msa.untile_routing_keys(cfg, KR).reshape(-1, d)[0].double()
    for got in (key, Vbar.reshape(d).double()):
        assert ((got - want).abs() <= 2.0 ** -8 * want).all()
    assert abs(float(inv.reshape(-1)[0]) * float(key.norm()) - 1) <= 2e-6


# (N, Hkv, r, G, d, B, M, k, Lloc, scope, rotated): many (query, KV head) pairs in the decode kernel
ATT_LINEAR = [
    (40, 8, 4, 512, 128, 20, 1, 18, 5, "group", 0),      # 160 pairs of 289 steps, three splits each
    (33, 8, 1, 512, 128, 45, 1, 20, 1791, "all", 0),     # 360 pairs of 376, two
    (25, 2, 2, 256, 64, 150, 2, 21, 130, "group", 0),    # 600 pairs of 173, one; two query tokens with selections of their own
    # the linear split, ranges that end inside pairs
    (40, 8, 4, 512, 128, 33, 1, 24, 430, "group", 0),    # 264 pairs of 398 steps in ranges of 416
    (40, 8, 1, 512, 128, 35, 1, 9, 170, "all", 0),       # 280 of 150 in 168: ranges meet three pairs
    (40, 8, 1, 512, 128, 33, 1, 24, 430, "all", 1),      # keys stored rotated
    (70, 8, 1, 8, 128, 39, 1, 64, 2880, "group", 1),     # the same, four documents per step: 312 of 106 in 136
    (30, 8, 1, 512, 64, 34, 1, 22, 1056, "group", 0),    # d = 64: 272 of 385 in 208
    (50, 4, 2, 256, 64, 68, 1, 44, 1056, "all", 1),
    (70, 8, 1, 16, 64, 34, 1, 64, 6976, "group", 1),     # 272 of 250 in 136
]


@pytest.mark.parametrize("N,Hkv,r,G,d,B,M,k,Lloc,scope,rotated", ATT_LINEAR)
def test_decode_attention_linear_split(N, Hkv, r, G, d, B, M, k, Lloc, scope, rotated):
    """Against the oracle on some queries, and every query against the same call with one query alone (another split);
    a pad and queries that see only a part of the local context among them."""
    say(f"linear split N={N} Hkv={Hkv} r={r} G={G} d={d} B={B} M={M} k={k} Lloc={Lloc} {scope} rotated={rotated}")
    cfg = msa.MsaConfig(N, G, G, Hkv * r, Hkv, d, 1e6, bank_keys_rotated=rotated,
                        select_scope=msa.MSA_SCOPE_ALL if scope == "all" else msa.MSA_SCOPE_GROUP)
    S_ = 1 if scope == "all" else Hkv
    Kb, K = S.normal_bf16(56000, (N, Hkv, G, d))
    Vb, V = S.normal_bf16(56001, (N, Hkv, G, d))
    qb, q = S.normal_bf16(56002, (B, M, Hkv * r, d))
    Klb, Kl = S.normal_bf16(56003, (B, Hkv, Lloc, d))
    Vlb, Vl = S.normal_bf16(56004, (B, Hkv, Lloc, d))
    rng = np.random.default_rng(56005)
    idx = np.argsort(rng.random((B, M, S_, N)), axis=-1)[..., :k].astype(np.int32)
    idx[:, :, :, k - 1] = -1
    q_pos = G + rng.integers(-1, Lloc, (B, M)).astype(np.int32)
    args = [dev(Kb), dev(Vb), torch.from_numpy(idx).cuda(), dev(Klb), dev(Vlb), G, torch.from_numpy(q_pos).cuda()]
    ws = torch.full((msa.sparse_attend_workspace_bytes(cfg, B, M, k, Lloc),), 0xA5, dtype=torch.uint8, device="cuda")
    dq = dev(qb)
    out, lse = msa.msa_sparse_attend(cfg, dq, *args, workspace=ws)
    again, lse2 = msa.msa_sparse_attend(cfg, dq, *args, workspace=ws)   # the arrival counters are ready for a replay
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), again.view(torch.int16)) and torch.equal(lse, lse2)
    for b in range(B):
        sl = slice(b, b + 1)
        one, l1 = msa.msa_sparse_attend(cfg, dq[sl].clone(), args[0], args[1], args[2][sl].clone(), args[3][sl].clone(),
                                        args[4][sl].clone(), G, args[6][sl].clone())
        torch.cuda.synchronize()
        # the same fp32 sums in another order, rounded to bf16 once: neighbours at most, which lie up to 2^-7 of the value
        # apart (8 significant bits, at the low end of a binade)
        x, y = out[b].float(), one[0].float()
        assert (x - y).abs().max() <= 2.0 ** -7 * y.abs().max() + 1e-6
        assert (lse[b] - l1[0]).abs().max() <= 1e-4
    for b in (0, B // 2, B - 1):
        oo, ol = O.sparse_attend(q[b:b + 1], K, V, idx[b:b + 1].astype(np.int64), Kl[b:b + 1], Vl[b:b + 1], G,
                                 q_pos[b:b + 1], 1e6, mem_rotated=bool(rotated))
        go = out[b:b + 1].float().cpu().numpy().astype(np.float64)
        assert np.abs(go - oo).max() <= 2e-2 and np.linalg.norm(go - oo) <= 5e-3 * np.linalg.norm(oo)
        assert np.allclose(lse[b:b + 1].cpu().numpy(), ol, rtol=0, atol=5e-3)


def attend_least(cfg, args, ws):
    """The least workspace size that a call accepts (sizes above it are all accepted)."""
    no, yes = 0, ws.numel()
    while yes - no > 1:
        mid = (no + yes) // 2
        try:
            msa.msa_sparse_attend(cfg, *args, workspace=ws[:mid])
            yes = mid
        except msa.MsaError as e:
            assert e.status == msa.MSA_ERR_WORKSPACE
            no = mid
    return yes


def docs_window(Hkv, r, G, d, S_, k, BM, tokens):
    """Workspace of the document-by-document path that grows with the tokens of a window."""
    up = lambda n: (n + 255) // 256 * 256
    steps, parts = G // 32, 1
    while parts < 4 and 2 * parts * k <= 128 and BM * k * Hkv * parts < 2048 and steps // (2 * parts) >= 4 and steps % (2 * parts) == 0:
        parts *= 2
    e, rows = S_ * tokens * k, tokens * Hkv * r
    return (up(rows * d * 4) + up(e * 16) + up(e * 4) + up(S_ * tokens * 4 << (k - 1).bit_length()) +
            up(rows * k * parts * d * 4) + up(rows * k * parts * 8))


# (N, Hkv, r, G, d, B, M, k, Lloc, scope, rotated, ragged): many tokens with selections of their own, document by document
ATT_DOCS = [
    (40, 2, 4, 128, 128, 1, 70, 30, 70, "group", 0, False),    # four tokens per item
    (24, 2, 8, 64, 128, 2, 64, 40, 40, "all", 0, True),        # two; one list for both heads
    (9, 3, 2, 256, 64, 1, 100, 16, 33, "group", 0, True),      # eight; nearly every document in every selection
    (30, 2, 1, 32, 64, 2, 100, 31, 32, "group", 0, False),     # sixteen; documents of one step
    (33, 2, 4, 1024, 128, 1, 16, 16, 300, "group", 0, True),   # few items: documents in four parts, some of them empty
    (50, 2, 4, 96, 128, 1, 50, 64, 64, "group", 1, False),     # keys stored rotated, the largest selection
    (50, 1, 8, 64, 64, 3, 64, 48, 50, "all", 1, True),
    (600, 8, 4, 64, 128, 1, 150, 20, 150, "group", 0, False),  # more than 64 items for one wave
    (13000, 1, 4, 32, 64, 1, 400, 32, 40, "group", 0, False),  # more documents than the sort counts in LDS
]


@pytest.mark.parametrize("N,Hkv,r,G,d,B,M,k,Lloc,scope,rotated,ragged", ATT_DOCS)
def test_attention_document_by_document(N, Hkv, r, G, d, B, M, k, Lloc, scope, rotated, ragged):
    """Against the oracle, with pads, ids outside the bank and a document listed twice; then with the smaller workspaces
    that the path takes: windows of tokens, whose results are the same bits; and with one byte less than the smallest of
    them and the least that is accepted, which the kernel that takes token by token serves, whose fp32 sums run in another
    order (one rounding to bf16: 2^-7 of the value)."""
    say(f"by document N={N} Hkv={Hkv} r={r} G={G} d={d} B={B} M={M} k={k} Lloc={Lloc} {scope} rot={rotated} ragged={ragged}")
    rng = np.random.default_rng(58005)
    lens = rng.integers(1, G + 1, N).astype(np.int32) if ragged else None
    cfg = msa.MsaConfig(N, G, G, Hkv * r, Hkv, d, 1e6, bank_keys_rotated=rotated,
                        doc_lens=torch.from_numpy(lens).cuda() if ragged else None,
                        select_scope=msa.MSA_SCOPE_ALL if scope == "all" else msa.MSA_SCOPE_GROUP)
    S_ = 1 if scope == "all" else Hkv
    Kb, K = S.normal_bf16(58000, (N, Hkv, G, d))
    Vb, V = S.normal_bf16(58001, (N, Hkv, G, d))
    qb, q = S.normal_bf16(58002, (B, M, Hkv * r, d))
    Klb, Kl = S.normal_bf16(58003, (B, Hkv, Lloc, d))
    Vlb, Vl = S.normal_bf16(58004, (B, Hkv, Lloc, d))
    idx = rng.integers(0, N, (B, M, S_, k)).astype(np.int32)          # documents twice in a selection among them
    idx[:, ::3, :, k - 1] = -1
    idx[:, 1::5, :, 0] = N + 3
    idx[0, 2] = -1                                                     # a token with the local context alone
    q_pos = (G + rng.integers(-1, Lloc, (B, M))).astype(np.int32)
    args = [dev(qb), dev(Kb), dev(Vb), torch.from_numpy(idx).cuda(), dev(Klb), dev(Vlb), G, torch.from_numpy(q_pos).cuda()]
    size = msa.sparse_attend_workspace_bytes(cfg, B, M, k, Lloc)
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
    out, lse = msa.msa_sparse_attend(cfg, *args, workspace=ws)
    torch.cuda.synchronize()
    oo, ol = O.sparse_attend(q, K, V, np.where(idx >= N, -1, idx).astype(np.int64), Kl, Vl, G, q_pos, 1e6,
                             lens=lens, mem_rotated=bool(rotated))
    go = out.float().cpu().numpy().astype(np.float64)
    assert np.abs(go - oo).max() <= 2e-2 and np.linalg.norm(go - oo) <= 5e-3 * np.linalg.norm(oo)
    seen = np.isfinite(ol)
    gl = lse.cpu().numpy()
    assert np.array_equal(np.isfinite(gl), seen) and np.abs(gl[seen] - ol[seen]).max() <= 5e-3
    least, BM = attend_least(cfg, args, ws), B * M
    up = lambda n: (n + 255) // 256 * 256
    path = least + up(S_ * N * 8) + up(S_ * N * 4) + up(S_ * 8)
    need = lambda tokens: path + docs_window(Hkv, r, G, d, S_, k, BM, tokens)
    assert need(BM) <= size
    several = uneven = 0
    for tokens in sorted({BM, BM - 1, BM // 2, 2 * BM // 5, 64} - set(range(min(64, BM))) - set(range(BM + 1, 65))):
        part = ws[:need(tokens)]
        part.fill_(0xFF)
        o2, l2 = msa.msa_sparse_attend(cfg, *args, workspace=part)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, l2), tokens
        n = -(-BM // tokens)
        several += n > 1
        uneven += BM % -(-BM // n) != 0
    assert several >= (BM > 64) and uneven >= (BM >= 200), (several, uneven)
    for bytes_ in (need(min(64, BM)) - 1, least):
        part = ws[:bytes_]
        part.fill_(0xFF)
        o2, l2 = msa.msa_sparse_attend(cfg, *args, workspace=part)
        torch.cuda.synchronize()
        assert not torch.equal(lse, l2)      # another order of the sums: the path was left
        x, y = o2.float(), out.float()
        assert (x - y).abs().max() <= 2.0 ** -7 * y.abs().max() + 1e-6
        assert (l2 - lse)[torch.isfinite(lse)].abs().max() <= 1e-4


@pytest.mark.parametrize("scope", ["group", "all"])
def test_attention_document_by_document_of_shared_selections(scope):
    """One selection for all tokens of a batch row over keys stored rotated (the tiled kernel takes raw keys alone): every
    document is shared by all of them; against the oracle and against tokens with copies of that selection."""
    N, Hkv, r, G, d, B, M, k, Lloc = 50, 2, 4, 96, 128, 2, 64, 16, 64
    say(f"by document, shared selections, {scope}")
    S_ = 1 if scope == "all" else Hkv
    scope_ = msa.MSA_SCOPE_ALL if scope == "all" else msa.MSA_SCOPE_GROUP
    cfg = msa.MsaConfig(N, G, G, Hkv * r, Hkv, d, 1e6, bank_keys_rotated=1, token_pool=1, select_scope=scope_)
    Kb, K = S.normal_bf16(58100, (N, Hkv, G, d))
    Vb, V = S.normal_bf16(58101, (N, Hkv, G, d))
    qb, q = S.normal_bf16(58102, (B, M, Hkv * r, d))
    Klb, Kl = S.normal_bf16(58103, (B, Hkv, Lloc, d))
    Vlb, Vl = S.normal_bf16(58104, (B, Hkv, Lloc, d))
    idx = np.random.default_rng(58105).integers(0, N, (B, 1, S_, k)).astype(np.int32)
    idx[:, :, :, 3] = -1
    q_pos = np.tile(G + np.arange(M, dtype=np.int32), (B, 1))
    tail = [dev(Klb), dev(Vlb), G, torch.from_numpy(q_pos).cuda()]
    out, lse = msa.msa_sparse_attend(cfg, dev(qb), dev(Kb), dev(Vb), torch.from_numpy(idx).cuda(), *tail)
    each = np.ascontiguousarray(np.broadcast_to(idx, (B, M, S_, k)))
    out2, lse2 = msa.msa_sparse_attend(cfg.replace(token_pool=0), dev(qb), dev(Kb), dev(Vb), torch.from_numpy(each).cuda(), *tail)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse, lse2)
    oo, ol = O.sparse_attend(q, K, V, idx.astype(np.int64), Kl, Vl, G, q_pos, 1e6, mem_rotated=True)
    go = out.float().cpu().numpy().astype(np.float64)
    assert np.abs(go - oo).max() <= 2e-2 and np.linalg.norm(go - oo) <= 5e-3 * np.linalg.norm(oo)
    assert np.abs(lse.cpu().numpy() - ol).max() <= 5e-3


@pytest.mark.parametrize("scope,r,k", [("all", 4, 8), ("group", 4, 16), ("group", 8, 8)])
def test_attention_document_by_document_of_pads(scope, r, k):
    """Selections without a document: the local context alone, against the oracle, from a workspace full of NaN; and sooner
    than with documents (128 documents shared by all; pads that were written out as empty partials by the one sorting
    workgroup of a list took up to five times as long)."""
    N, Hkv, G, d, B, M, Lloc = 128, 8, 512, 128, 1, 100, 100
    say(f"by document, pads, {scope} r={r} k={k}")
    S_ = 1 if scope == "all" else Hkv
    cfg = msa.MsaConfig(N, G, G, Hkv * r, Hkv, d, 1e6, select_scope=msa.MSA_SCOPE_ALL if scope == "all" else msa.MSA_SCOPE_GROUP)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(58200)
    K, V = (torch.randn((N, Hkv, G, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    qb, q = S.normal_bf16(58201, (B, M, Hkv * r, d))
    Klb, Kl = S.normal_bf16(58202, (B, Hkv, Lloc, d))
    Vlb, Vl = S.normal_bf16(58203, (B, Hkv, Lloc, d))
    q_pos = (G + np.arange(M, dtype=np.int32)).reshape(B, M)
    some = torch.rand((B, M, S_, N), generator=gen, device="cuda").topk(k, dim=-1).indices.to(torch.int32)
    none = torch.full_like(some, -1)
    none[:, :, :, ::2] = N
    ws = torch.empty(msa.sparse_attend_workspace_bytes(cfg, B, M, k, Lloc), dtype=torch.uint8, device="cuda")
    dq, dKl, dVl, dpos = dev(qb), dev(Klb), dev(Vlb), torch.from_numpy(q_pos).cuda()
    took = []
    for idx in (some, none):
        ws.fill_(0xFF)
        out, lse = msa.msa_sparse_attend(cfg, dq, K, V, idx, dKl, dVl, G, dpos, workspace=ws)
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                msa.msa_sparse_attend(cfg, dq, K, V, idx, dKl, dVl, G, dpos, out, lse, ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
    oo, ol = O.sparse_attend(q, np.zeros((1, Hkv, G, d)), np.zeros((1, Hkv, G, d)), np.full((B, M, S_, k), -1, dtype=np.int64), Kl, Vl,
                             G, q_pos, 1e6)
    go = out.float().cpu().numpy().astype(np.float64)
    assert np.abs(go - oo).max() <= 2e-2 and np.linalg.norm(go - oo) <= 5e-3 * np.linalg.norm(oo)
    assert np.abs(lse.cpu().numpy() - ol).max() <= 5e-3
    assert took[1] < took[0], took


# (N, Hkv, r, G, d, B, M, k, Lloc, scope, rotated, ragged): no document in two selections, so that an item is a chain of a
# token's documents, of up to ...
ATT_CHAINS = [
    (1600, 4, 2, 64, 64, 1, 96, 16, 96, "group", 0, False),     # ... four
    (800, 8, 4, 64, 64, 1, 128, 6, 40, "group", 0, True),       # ... three, two per token
    (1600, 2, 8, 64, 128, 1, 128, 12, 50, "all", 1, True),      # ... two; items of two tokens were they shared
    (1600, 4, 1, 64, 64, 2, 48, 16, 32, "group", 1, True),      # ... four; of sixteen
    (300, 4, 2, 2048, 128, 1, 32, 8, 33, "group", 0, True),     # ... one, the documents in two parts
    (13000, 1, 4, 32, 64, 1, 800, 16, 40, "group", 0, False),   # counters in memory, documents looked up again by every phase
    (530000, 1, 4, 32, 64, 1, 400, 32, 40, "group", 0, False),  # ... more documents than have a bit in LDS
]


@pytest.mark.parametrize("N,Hkv,r,G,d,B,M,k,Lloc,scope,rotated,ragged", ATT_CHAINS)
def test_attention_of_selections_without_common_documents(N, Hkv, r, G, d, B, M, k, Lloc, scope, rotated, ragged):
    """With pads, ids outside the bank, tokens with one document and with none, from workspaces full of NaN: against the
    oracle (small documents), and against the kernel that takes token by token, whose fp32 sums run in another order (one
    rounding to bf16: 2^-7 of the value)."""
    say(f"chains N={N} Hkv={Hkv} r={r} G={G} d={d} B={B} M={M} k={k} Lloc={Lloc} {scope} rot={rotated} ragged={ragged}")
    rng = np.random.default_rng(58300 + N)
    lens = rng.integers(1, G + 1, N).astype(np.int32) if ragged else None
    cfg = msa.MsaConfig(N, G, G, Hkv * r, Hkv, d, 1e6, bank_keys_rotated=rotated,
                        doc_lens=torch.from_numpy(lens).cuda() if ragged else None,
                        select_scope=msa.MSA_SCOPE_ALL if scope == "all" else msa.MSA_SCOPE_GROUP)
    S_ = 1 if scope == "all" else Hkv
    gen = torch.Generator(device="cuda")
    gen.manual_seed(58300)
    K, V = (torch.empty((N, Hkv, G, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(2))
    qb, q = S.normal_bf16(58301, (B, M, Hkv * r, d))
    Klb, Kl = S.normal_bf16(58302, (B, Hkv, Lloc, d))
    Vlb, Vl = S.normal_bf16(58303, (B, Hkv, Lloc, d))
    idx = np.stack([rng.permutation(N)[:B * M * k].reshape(B, M, k) for _ in range(S_)], axis=2).astype(np.int32)
    idx[:, ::3, :, k // 2] = -1
    idx[:, 1::5, :, 0] = N + 3
    idx[0, 2] = -1
    idx[0, 5, :, 1:] = -1
    idx[0, 7, :, :k - 1] = -1
    q_pos = (G + rng.integers(-1, Lloc, (B, M))).astype(np.int32)
    args = [dev(qb), K, V, torch.from_numpy(idx).cuda(), dev(Klb), dev(Vlb), G, torch.from_numpy(q_pos).cuda()]
    ws = torch.empty(msa.sparse_attend_workspace_bytes(cfg, B, M, k, Lloc), dtype=torch.uint8, device="cuda")
    least = attend_least(cfg, args, ws)
    assert least < ws.numel()
    ws.fill_(0xFF)
    out, lse = msa.msa_sparse_attend(cfg, *args, workspace=ws)
    torch.cuda.synchronize()
    up = lambda n: (n + 255) // 256 * 256
    flags = least + up(S_ * N * 8) + up(S_ * N * 4)
    assert (ws[flags + 4 * S_:flags + 8 * S_].view(torch.int32) == 1).all()      # every list in chains
    if B * M > 64:   # windows of tokens: the same bits
        part = ws[:flags + up(S_ * 8) + docs_window(Hkv, r, G, d, S_, k, B * M, 70)]
        part.fill_(0xFF)
        o2, l2 = msa.msa_sparse_attend(cfg, *args, workspace=part)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, l2)
    ws.fill_(0xFF)
    o2, l2 = msa.msa_sparse_attend(cfg, *args, workspace=ws[:least])
    torch.cuda.synchronize()
    x, y = o2.float(), out.float()
    assert torch.isfinite(y).all() and (x - y).abs().max() <= 2.0 ** -7 * y.abs().max() + 1e-6
    seen = torch.isfinite(l2)
    assert torch.equal(torch.isfinite(lse), seen) and (l2 - lse)[seen].abs().max() <= 1e-4
    if N * G > 1 << 18:
        return
    to64 = lambda t: t.float().cpu().numpy().astype(np.float64)
    oo, ol = O.sparse_attend(q, to64(K), to64(V), np.where(idx >= N, -1, idx).astype(np.int64), Kl, Vl, G, q_pos, 1e6,
                             lens=lens, mem_rotated=bool(rotated))
    go = to64(out)
    assert np.abs(go - oo).max() <= 2e-2 and np.linalg.norm(go - oo) <= 5e-3 * np.linalg.norm(oo)
    seen = np.isfinite(ol)
    assert np.abs(lse.cpu().numpy()[seen] - ol[seen]).max() <= 5e-3
