"""The routed layers of a Memory Sparse Attention model as one per-token loop over the C-ABI entry points.

Section 3.2.1 applies routing in the latter half of the model's layers; Section 3.4.2 keeps, for every routed layer,
the routing keys in device memory and the pooled content bank (K-bar, V-bar) either in device memory or, tiered, in
host DRAM from which the selected documents are fetched.  A LayerStack holds those per-layer banks and runs, for one
batch of query tokens, score + top-k -> (fetch) -> attention in every layer.  Where the banks are in device memory a step
runs on the caller's stream, its attention on a second one where that pays; with host banks scoring runs on one stream
and fetch + attention on another.  With two streams layer l + 1 is routed while layer l's winners are still being fetched
and attended (the layers' queries are inputs here; in a model they come out of the layer below, which orders the streams
the same way through events).

Orchestration only: every step of the path runs in the library's kernels.
"""
import torch

from . import (MSA_ERR_HIP, MsaConfig, MsaError, msa_build_routing_keys, msa_fetch_selected, msa_layers_step,
               msa_pool_kv, msa_score_topk, msa_sparse_attend, score_topk_workspace_bytes, sparse_attend_workspace_bytes,
               alloc_routing_index, fetch_slots)


def attention_beside_routing(n_layers, queries, index_bytes):
    """Whether a step with every bank in device memory puts attention on a second stream, beside the next layer's scan.

    The second stream costs about 13 us per step for its hand-over, and every layer but the last wins some of its attention
    back: the more, the longer the scans and the more queries.  Measured over 150 shapes, us per step on one stream / on two
    (8 heads of 128, 16 documents, 1024 local rows; n layers of x MB, q queries): 2 of 56 to 937, 1 to 16 q: 74 / 87 to 543 /
    553; 3 of 93, 4 q 133 / 134; 3 of 187, 8 q 214 / 203; 4 of 31, 1 q 133 / 147; 4 of 56, 1 q 142 / 148, 8 q 169 / 157; 4 of
    128, 1 q 199 / 190, 16 q 256 / 239; 4 of 1525, 8 q 1149 / 1128; 6 of 31, 8 q 234 / 214; 8 of 16, 1 q 231 / 260, 8 q 280 /
    262; 18 of 23, 8 q 673 / 531.  The rule is at most 2 % from the better way there, and at most 4.4 % over 30 shapes with
    longer attention, where a few workgroups more or less decide (16 q, 4096 local rows: 4 of 78 351 / 366, 4 of 128 385 / 397;
    2048 rows, 32 documents: 4 of 64 258 / 265, 4 of 93 280 / 273)."""
    return index_bytes * (n_layers - 2) >= (64 if queries >= 8 else 128) << 20


class LayerStack:
    def __init__(self, cfg, n_layers, B, M, k, Lloc, tier="hbm", device="cuda"):
        """cfg: the config of the un-pooled bank (N documents of G tokens, chunk P).  tier: "hbm" keeps every
        layer's pooled bank in device memory, "host" in pinned host memory (fetched per step)."""
        assert tier in ("hbm", "host")
        self.cfg, self.L, self.B, self.M, self.k, self.Lloc, self.tier, self.dev = cfg, n_layers, B, M, k, Lloc, tier, device
        C = cfg.chunks_per_doc
        # the pooled bank is a bank of N documents of C rows whose keys carry their positions
        self.pcfg = MsaConfig(cfg.n_docs, C, C, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.rope_base,
                              sim=cfg.sim, select_scope=cfg.select_scope, token_pool=cfg.token_pool,
                              bank_keys_rotated=1)
        self.KR, self.inv, self.Kbar, self.Vbar = [], [], [], []
        shape = (cfg.n_docs, cfg.n_kv_heads, C, cfg.head_dim)
        for _ in range(n_layers):
            kr, inv = alloc_routing_index(cfg, device)
            self.KR.append(kr)
            self.inv.append(inv)
            if tier == "hbm":
                self.Kbar.append(torch.empty(shape, dtype=torch.bfloat16, device=device))
                self.Vbar.append(torch.empty(shape, dtype=torch.bfloat16, device=device))
        if tier == "host":
            # As many distinct pooled banks as the machine lets this process pin (at least one); when that is
            # fewer than n_layers, layer l reads bank l % n_banks -- the same bytes travel per layer, which is what
            # a timing needs; a model needs every layer's own bank.
            for l in range(n_layers):
                try:
                    kb = torch.empty(shape, dtype=torch.bfloat16, pin_memory=True)
                    vb = torch.empty(shape, dtype=torch.bfloat16, pin_memory=True)
                except RuntimeError:
                    if l == 0:
                        raise
                    break
                self.Kbar.append(kb)
                self.Vbar.append(vb)
        self.n_banks = len(self.Kbar)
        m_sel = 1 if cfg.token_pool else M
        n_sel = 1 if cfg.select_scope == 1 else cfg.n_kv_heads
        self.idx = [torch.empty((B, m_sel, n_sel, k), dtype=torch.int32, device=device) for _ in range(n_layers)]
        self.val = [torch.empty((B, m_sel, n_sel, k), dtype=torch.float32, device=device) for _ in range(n_layers)]
        self.ws_s = torch.empty(score_topk_workspace_bytes(cfg, B, M, k), dtype=torch.uint8, device=device)
        self.acfg = self.pcfg
        if tier == "host":
            n_slots = fetch_slots(self.pcfg, B, M, k)
            self.K_stage = torch.empty((n_slots, cfg.n_kv_heads, C, cfg.head_dim), dtype=torch.bfloat16, device=device)
            self.V_stage = torch.empty_like(self.K_stage)
            self.idx_stage = torch.empty_like(self.idx[0])
            self.acfg = self.pcfg.replace(n_docs=n_slots)
        self.ws_a = torch.empty(sparse_attend_workspace_bytes(self.acfg, B, M, k, Lloc), dtype=torch.uint8, device=device)
        # (The "hbm" tier routes on the caller's stream.  s_route is made, and used once below, all the same: the four hardware
        # queues go round the streams as they are first used, and an s_attend on the caller's queue runs no work beside it.
        # Four layers of 197 MB, 12 queries, the sixth stack of a program: 293 us with the pair, 350 with s_attend alone, 317 on
        # one stream.)
        self.s_route, self.s_attend = torch.cuda.Stream(device), torch.cuda.Stream(device)
        self.two_streams = attention_beside_routing(n_layers, B * M, self.KR[0].numel() * 2)
        self.last_id = None   # torch's number of the stream that the last step of the "hbm" tier was called on
        self.ev_scored = [torch.cuda.Event() for _ in range(n_layers)]
        self.ev_fork, self.ev_join, self.ev_captured = torch.cuda.Event(), torch.cuda.Event(), torch.cuda.Event()
        for ev in self.ev_scored + [self.ev_fork, self.ev_join, self.ev_captured]:
            ev.record(self.s_route)   # an event exists from its first record on

    # ---- offline stage (Section 3.4.1, Stage 1), one layer at a time; K and V may be the same buffer refilled ----
    def set_layer_keys(self, layer, K):
        """Routing index and pooled, position-encoded key bank of one layer from its keys K [N][Hkv][G][d]."""
        msa_build_routing_keys(self.cfg, K, KR=self.KR[layer], inv_norm=self.inv[layer])
        if layer >= self.n_banks:
            return
        if self.tier == "hbm":
            msa_pool_kv(self.cfg, K, None, Kbar=self.Kbar[layer])
        else:
            tmp, _ = msa_pool_kv(self.cfg, K, None)
            self.Kbar[layer].copy_(tmp)

    def set_layer_values(self, layer, V):
        if layer >= self.n_banks:
            return
        if self.tier == "hbm":
            msa_pool_kv(self.cfg, None, V, Vbar=self.Vbar[layer])
        else:
            _, tmp = msa_pool_kv(self.cfg, None, V)
            self.Vbar[layer].copy_(tmp)

    def bytes(self):
        index = sum(t.numel() * 2 for t in self.KR) + sum(t.numel() * 4 for t in self.inv)
        bank = sum(t.numel() * 2 for t in self.Kbar) + sum(t.numel() * 2 for t in self.Vbar)
        return index, bank

    # ---- online: one batch of query tokens through every routed layer --------------------------------------
    def step(self, qs, Klocs, Vlocs, pos0, q_pos, outs, lses, overlap=True):
        """qs[l] bf16 [B][M][Hq][d]: the routing/attention query of layer l; Klocs[l], Vlocs[l] its local cache;
        outs[l], lses[l] receive its attention output (None: not wanted).  overlap=False runs everything on one stream.
        One host thread at a time: the stack's workspaces, selections and events are shared by its steps.  Steps of the
        "hbm" tier from different streams follow each other; replays of a captured step are ordered by whoever replays it."""
        cur = torch.cuda.current_stream(self.dev)
        if self.tier == "hbm":
            # Routing runs on the caller's stream: handed to a stream of its own and joined again, small steps waited more
            # than they worked (two layers, 1000 documents, 5 queries 87 us -> 62; four, 256 documents, 2 queries 141 -> 95).
            # Steps from different streams follow each other all the same, since they share the workspaces: each waits for
            # the event at the end of the step before (nothing else that its stream holds, and no stream is kept).
            capturing = torch.cuda.is_current_stream_capturing()
            join = self.ev_captured if capturing else self.ev_join
            if not capturing:
                # the same stream again has the end of that step ahead of it (a second wait is 4 us with two streams); but one
                # that is not torch's own may be a new one in the place of one that was destroyed
                own = cur.cuda_stream == 0 or cur.stream_id != cur.cuda_stream
                if not own or cur.stream_id != self.last_id:
                    cur.wait_event(self.ev_join)
                self.last_id = cur.stream_id if own else None
            s_a = self.s_attend if overlap and self.two_streams else cur
            # the whole step in one native call: as single calls from here the host was the bound of small steps (four
            # layers, 557 documents, 5 streams: 223 us -> 153; two layers, 956 documents, 2 streams: 141 -> 93)
            try:
                msa_layers_step(self.cfg, self.acfg,
                                [(qs[l], self.KR[l], self.inv[l], self.idx[l], self.val[l], self.Kbar[l], self.Vbar[l],
                                  Klocs[l], Vlocs[l], torch.empty_like(qs[l]) if outs[l] is None else outs[l], lses[l],
                                  self.ev_scored[l]) for l in range(self.L)],
                                self.k, pos0, q_pos, self.ws_s, self.ws_a, cur, cur, s_a, self.ev_fork, join)
            except MsaError as e:
                if e.status == MSA_ERR_HIP and not capturing:   # part of the step may run: the caller's stream awaits it
                    join.record(cur)
                raise
            return
        s_r = self.s_route
        s_a = self.s_attend if overlap else s_r
        s_r.wait_stream(cur)
        if overlap:
            s_a.wait_stream(cur)
        for l in range(self.L):
            msa_score_topk(self.cfg, qs[l], self.KR[l], self.inv[l], self.k, self.idx[l], self.val[l], self.ws_s,
                           stream=s_r)
            if overlap:
                self.ev_scored[l].record(s_r)
                s_a.wait_event(self.ev_scored[l])
            msa_fetch_selected(self.pcfg, self.Kbar[l % self.n_banks], self.Vbar[l % self.n_banks], self.idx[l], self.B, self.M, self.K_stage,
                               self.V_stage, self.idx_stage, stream=s_a)
            msa_sparse_attend(self.acfg, qs[l], self.K_stage, self.V_stage, self.idx_stage, Klocs[l], Vlocs[l],
                              pos0, q_pos, outs[l], lses[l], self.ws_a, stream=s_a)
        cur.wait_stream(s_r)
        if overlap:
            cur.wait_stream(s_a)
