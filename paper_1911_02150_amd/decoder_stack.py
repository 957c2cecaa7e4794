"""Incremental decoding of a decoder-only stack whose attention is the library's
multi-query (or multi-head) decode step.  Pure glue: every operation is a call
into the HIP library; torch only holds the device buffers.

Stack (the model family of the paper's Section 4.1, random weights): token
embedding + learned positional embedding; per layer  x += Attn(LN(x)),
x += relu(LN(x) W1) W2;  final LN; logits = x E^T (embedding tied to the output
layer); no biases; layernorm gain 1, bias 0, eps 1e-6.

Nothing is kept of the weights but the tensors themselves: a pass multiplies by what they hold when it runs, called or
replayed from a graph (a graph reads the tensors that it was captured with).
"""
from __future__ import annotations

import torch

from . import binding as B


class DecoderStack:
    def __init__(self, weights: dict, batch: int, cap: int, multi_head: bool, device="cuda:0",
                 cache_dtype=torch.bfloat16):
        dev = torch.device(device)
        self.dev, self.b, self.cap, self.multi_head = dev, batch, cap, multi_head
        self.E = torch.from_numpy(weights["E"]).to(dev)
        self.pos = torch.from_numpy(weights["pos"]).to(dev)
        self.layers = [{k: torch.from_numpy(v).to(dev) for k, v in lw.items()} for lw in weights["layers"]]
        h, d, k = self.layers[0]["P_q"].shape
        v = self.layers[0]["P_o"].shape[2]
        self.h, self.d, self.k, self.v = h, d, k, v
        self._parts = {}
        kshape = (batch, h, cap, k) if multi_head else (batch, cap, k)
        vshape = (batch, h, cap, v) if multi_head else (batch, cap, v)
        self.K = [torch.zeros(kshape, dtype=cache_dtype, device=dev) for _ in self.layers]
        self.V = [torch.zeros(vshape, dtype=cache_dtype, device=dev) for _ in self.layers]
        self.lens = [torch.zeros(batch, dtype=torch.int32, device=dev) for _ in self.layers]
        self._lens_next = [torch.zeros(batch, dtype=torch.int32, device=dev) for _ in self.layers]

    # -- pieces, so that a test can look between them
    def embed(self, tokens: torch.Tensor, t: int) -> torch.Tensor:
        positions = torch.full((self.b,), t, dtype=torch.int32, device=self.dev)
        return B.mqa_stack_embed(tokens.to(torch.int32), positions, self.E, self.pos)

    def attention_append(self, l: int, x: torch.Tensor):
        """LN, projections of q and the new K/V rows, append.  Returns q and the float32 rows."""
        w = self.layers[l]
        hx = B.mqa_stack_layernorm(x)
        q = B.mqa_project_qkvo(B.MQA_PROJ_Q, hx, w["P_q"])
        mode = B.MQA_PROJ_KV_MH if self.multi_head else B.MQA_PROJ_KV
        kn = B.mqa_project_qkvo(mode, hx, w["P_k"])
        vn = B.mqa_project_qkvo(mode, hx, w["P_v"])
        B.mqa_append_kv(self.K[l], self.V[l], kn, vn, self.lens[l])
        return q, kn, vn

    def attention_append_fused(self, l: int, x: torch.Tensor) -> torch.Tensor:
        """LN, then q and the append of the new K/V rows in one launch.  Returns q."""
        return self._append_fused(l, B.mqa_stack_layernorm(x))

    def _append_fused(self, l: int, hx: torch.Tensor) -> torch.Tensor:
        w = self.layers[l]
        q = B.mqa_project_append_qkv(hx, w["P_q"], w["P_k"], w["P_v"], self.K[l], self.V[l], self.lens[l],
                                     self._lens_next[l])
        self.lens[l], self._lens_next[l] = self._lens_next[l], self.lens[l]      # the lengths alternate between two arrays
        return q

    def attention_attend(self, l: int, q: torch.Tensor) -> torch.Tensor:
        """Attention over the cache and the output projection.  Returns y."""
        dec = B.mha_decode_step if self.multi_head else B.mqa_decode_step
        o = dec(q, self.K[l], self.V[l], self.lens[l])
        return B.mqa_project_qkvo(B.MQA_PROJ_O, o, self.layers[l]["P_o"])

    def feed_forward(self, l: int, x: torch.Tensor) -> torch.Tensor:
        w = self.layers[l]
        hx = B.mqa_stack_layernorm(x)
        u = B.mqa_project_qkvo(B.MQA_PROJ_LINEAR, hx, w["W1"])
        B.mqa_stack_relu(u)
        return B.mqa_project_qkvo(B.MQA_PROJ_LINEAR, u, w["W2"])

    def logits(self, x: torch.Tensor) -> torch.Tensor:
        return self._logits(B.mqa_stack_layernorm(x))

    def _logits(self, hx: torch.Tensor) -> torch.Tensor:
        return B.mqa_project_qkvo(B.MQA_PROJ_O, hx.view(self.b, 1, self.d), self.E.view(1, -1, self.d))

    def _workspace(self, rows: int, nbytes: int = 0) -> torch.Tensor:
        """Scratch memory for the calls of one pass over `rows` rows, one after another on its stream (a pass's own: calls on several
        streams do not share it), nbytes at least."""
        cap = max(V.shape[-2] for V in self.V) if rows == self.b else 0        # (a step's attention; a program may have put other caches in)
        key = rows, cap, self.K[0].dtype
        known = self._parts.get(key)           # (a decoding loop asks for the same rows again and again: 1.5 us of a step)
        if known is None:
            sizes = [16, B.mqa_project_add_layernorm_workspace_bytes(B.MQA_PROJ_O, rows, self.d, self.h, self.v)]
            for ff in {w["W1"].shape[1] for w in self.layers}:
                sizes.append(B.mqa_project_add_layernorm_workspace_bytes(B.MQA_PROJ_LINEAR, rows, ff, 1, self.d))
            if cap:
                dt = B._cache_dtype(self.K[0])
                sizes.append(B.mqa_decode_workspace_bytes_default(self.b, self.h, cap, self.k, self.v, dt, self.multi_head))
            if len(self._parts) >= 16:
                self._parts.clear()
            known = self._parts[key] = max(sizes)
        return torch.empty(max(known, nbytes), dtype=torch.uint8, device=self.dev)

    # -- one decoding step for the whole stack: per layer 7 launches (fused q/K/V + append, attention (+ merge), output
    #    projection in parts, their sum added into x with the layernorm, W1 with relu, W2 in parts, the same)
    def step(self, tokens: torch.Tensor, t: int) -> torch.Tensor:
        x = self.embed(tokens, t)
        dec = B.mha_decode_step if self.multi_head else B.mqa_decode_step
        ws = self._workspace(self.b)
        hx = B.mqa_stack_layernorm(x)
        for l, w in enumerate(self.layers):
            q = self._append_fused(l, hx)
            o = dec(q, self.K[l], self.V[l], self.lens[l], workspace=ws)
            B.mqa_project_add_layernorm(B.MQA_PROJ_O, o, w["P_o"], x, out=hx, workspace=ws)
            u = B.mqa_project_qkvo_ex(B.MQA_PROJ_LINEAR, hx, w["W1"], epilogue=B.MQA_EPI_RELU)
            B.mqa_project_add_layernorm(B.MQA_PROJ_LINEAR, u, w["W2"], x, out=hx, workspace=ws)
        return self._logits(hx)

    def _prompt_workspace(self, b: int, n: int):
        """The workspace of a prompt's pass, and of which layers it holds the feed-forward in one call (without memory for it: of none)."""
        rows = b * n
        kv_rows = B.mqa_project_kv_workspace_bytes(b, n, self.d, 1, self.k, self.v, B._cache_dtype(self.K[0]))
        widths = [w["W1"].shape[1] for w in self.layers[:-1]]
        plans = {ff: B.mqa_stack_feed_forward_plan(rows, self.d, ff) for ff in set(widths)}
        in_one = [bool(plans[ff][0] & 1) for ff in widths]
        if any(in_one):
            try:
                return self._workspace(rows, max(kv_rows, *(nbytes for plan, nbytes in plans.values() if plan & 1))), in_one
            except torch.OutOfMemoryError:
                in_one = [False] * len(in_one)
        return self._workspace(rows, kv_rows), in_one

    # -- a whole prompt at once (multi-query only): bulk append + fused causal attention per layer
    def prefill(self, prompts: torch.Tensor) -> torch.Tensor:
        """prompts [b,n] int32, caches empty.  Returns the logits of the last prompt position [b,vocab]."""
        if self.multi_head:
            raise NotImplementedError("prefill is built for the multi-query cache")
        b, n = prompts.shape
        rows = b * n
        positions = torch.arange(n, dtype=torch.int32, device=self.dev).repeat(b)
        x = B.mqa_stack_embed(prompts.reshape(-1).to(torch.int32).contiguous(), positions, self.E, self.pos)   # [b*n,d]
        ws, in_one = self._prompt_workspace(b, n)
        hx = B.mqa_stack_layernorm(x)
        end = len(self.layers) - 1
        for l, w in enumerate(self.layers):
            if self.k % 16 == 0 and self.v % 16 == 0:
                now = self._lens_next[l]
                B.mqa_project_append_kv_rows(hx.view(b, n, self.d), w["P_k"], w["P_v"], self.K[l], self.V[l], self.lens[l], now,
                                             workspace=ws)
            else:
                now = self.lens[l]
                kn = B.mqa_project_qkvo(B.MQA_PROJ_KV, hx, w["P_k"]).view(b, n, self.k)
                vn = B.mqa_project_qkvo(B.MQA_PROJ_KV, hx, w["P_v"]).view(b, n, self.v)
                B.mqa_append_kv_rows(self.K[l], self.V[l], kn, vn, self.lens[l])
            if l == end:
                # Of the last layer, behind its K and V rows, only the last positions lead to a result, and each depends on itself and the
                # caches alone: the rest of the layer is a step's (six layers, b=128, n=128, d=1024, ff=4096: 6260 -> 5270 us)
                x, hx = (t.view(b, n, self.d)[:, n - 1].contiguous() for t in (x, hx))
                rows, ws = b, self._workspace(b)
            q = B.mqa_project_qkvo(B.MQA_PROJ_Q, hx, w["P_q"]).view(b, rows // b, self.h, self.k)
            o = B.mqa_prefill_attention(q, self.K[l], self.V[l], now, workspace=ws).view(rows, self.h, self.v)
            if l < end and in_one[l]:
                B.mqa_project_qkvo_ex(B.MQA_PROJ_O, o, w["P_o"], out=x, epilogue=B.MQA_EPI_ADD)
                B.mqa_stack_feed_forward(x, w["W1"], w["W2"], ws)
                B.mqa_stack_layernorm(x, out=hx)
                continue
            B.mqa_project_add_layernorm(B.MQA_PROJ_O, o, w["P_o"], x, out=hx, workspace=ws)
            u = B.mqa_project_qkvo_ex(B.MQA_PROJ_LINEAR, hx, w["W1"], epilogue=B.MQA_EPI_RELU)
            if l < end:
                B.mqa_project_add_layernorm(B.MQA_PROJ_LINEAR, u, w["W2"], x, out=hx, workspace=ws)
            else:                             # (logits() normalises)
                B.mqa_project_qkvo_ex(B.MQA_PROJ_LINEAR, u, w["W2"], out=x, epilogue=B.MQA_EPI_ADD)
        if now is not self.lens[-1]:      # the lengths advance in the arrays they are in: a caller may hold them
            torch._foreach_copy_(self.lens, self._lens_next)
        return self.logits(x)

    def greedy(self, logits: torch.Tensor) -> torch.Tensor:
        return B.mqa_stack_argmax(logits)
