"""Incremental decoding of a decoder-only stack whose attention is the library's
multi-query (or multi-head) decode step.  Pure glue: every operation is a call
into the HIP library; torch only holds the device buffers.

Stack (the model family of the paper's Section 4.1, random weights): token
embedding + learned positional embedding; per layer  x += Attn(LN(x)),
x += relu(LN(x) W1) W2;  final LN; logits = x E^T (embedding tied to the output
layer); no biases; layernorm gain 1, bias 0, eps 1e-6.
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
        self._exponent = B.load_library().mqa_stack_layernorm_exponent(d)
        self.pack()

    # -- packed weights (see mqa.h): laid out once, and again by themselves when a weight has been replaced or changed through torch.  A program
    #    that changes one behind torch's back, or wants a captured pass to see a change, calls pack(): the copies stay where they are.
    def pack(self):
        old = getattr(self, "_packs", {})
        self._packs, self._plans = {}, {}
        weights = list(self._packable())
        if self.dev.type != "cuda" or self.d % 32 or self.d > 4096 or any(t.is_inference() for _, _, t in weights):      # (no versions to tell a change by)
            return
        with torch.cuda.device(self.dev):
            self._pack(weights, old)

    def _pack(self, weights, old):
        for key, mode, t in weights:
            C, lines = t.shape
            before = self._packs.get((key[0], "W1")) if key[1] == "W2" else None
            if lines % 8 or C % 32 or t.shape[-1] % 8 or not t.is_contiguous() or t.dtype != torch.float32 or t.device != self.K[0].device or \
                    t.data_ptr() % 16 or (key[1] == "W2" and before is None) or B.load_library().mqa_stack_packed_bytes(lines, C, 1) == 0:
                continue
            p = old[key][0] if key in old and (old[key][0].N, old[key][0].C) == (lines, C) else None
            if p is None:
                p = B.PackedWeights(mode, t, before and before[0])
            else:
                p.row_scale = before and before[0]
                p.pack(t)
            self._packs[key] = p, t, t._version
        if self._packs:
            bad = torch.cat([p.verdict for p, _, _ in self._packs.values()]).tolist()
            self._unheld = {key for key, b in zip(self._packs, bad) if b}

    def _packable(self):
        for l, w in enumerate(self.layers):
            yield (l, "W1"), B.MQA_PROJ_LINEAR, w["W1"]
            yield (l, "W2"), B.MQA_PROJ_LINEAR, w["W2"]

    def _fresh(self) -> bool:
        return all(self.layers[l][name] is t and t._version == version for (l, name), (_, t, version) in self._packs.items())

    def _plan(self, rows: int):
        """How the products of a pass over `rows` rows run from packed weights (mqa_stack_product_plan; 0: they do not): per layer W1's,
        W2's and a last W2's without a layernorm behind it."""
        if not self._fresh():
            if torch.cuda.is_current_stream_capturing():      # (the packing asks the device: this pass goes without)
                return [(0, 0, 0)] * len(self.layers)
            self.pack()
        plan = self._plans.get(rows)
        if plan is None:
            def form(key, n, residual=False):
                return self._packs[key][0].plan(n, residual) if key in self._packs and key not in self._unheld else 0
            plan = []
            for l in range(len(self.layers)):
                w1 = form((l, "W1"), rows)
                plan.append((w1, w1 and form((l, "W2"), rows, True), w1 and form((l, "W2"), rows)))
            if len(self._plans) >= 16:             # (prompts of many lengths)
                self._plans.clear()
            self._plans[rows] = plan
        return plan

    def _packed_rows(self, rows: int, C: int) -> torch.Tensor:
        return torch.empty(4 * rows * C, dtype=torch.uint8, device=self.dev)

    def _hidden(self, l: int, hx, rows: int, form: int, next_form: int):
        """relu(hx W1): float32, or packed for the W2 that is."""
        if not form:
            return B.mqa_project_qkvo_ex(B.MQA_PROJ_LINEAR, hx, self.layers[l]["W1"], epilogue=B.MQA_EPI_RELU)
        W1 = self._packs[l, "W1"][0]
        if not next_form:
            u = torch.empty((rows, W1.N), dtype=torch.float32, device=self.dev)
            return B.mqa_stack_product(hx, W1, 2.0 ** -self._exponent, u, rows, form, B.MQA_EPI_RELU)
        # |hx 2^e . W1| <= sqrt(d) 2^e sqrt(d) 2^15 (the columns' largest values are below 2^15), and sqrt(d) 2^e <= 2^15: to 2^15 at most
        return B.mqa_stack_product(hx, W1, 2.0 ** (self._exponent - 30), self._packed_rows(rows, W1.N), rows, form, B.MQA_EPI_RELU_PACKED)

    def _add_hidden(self, l: int, u, out: torch.Tensor, rows: int, form: int, epilogue: int):
        B.mqa_stack_product(u, self._packs[l, "W2"][0], 2.0 ** (30 - 2 * self._exponent), out, rows, form, epilogue)

    def _feed_forward(self, l: int, plan, hx, x: torch.Tensor, ws: torch.Tensor, out, packed):
        """x += relu(hx W1) W2 with hx packed or not, by the plan; then the layernorm of x to out and packed (either may be None)."""
        w1, w2, _ = plan
        u = self._hidden(l, hx, x.shape[0], w1, w2)
        if not w2:
            self._project_norm(B.MQA_PROJ_LINEAR, u, self.layers[l]["W2"], x, ws, out, packed)
        elif w2 & 15 == 1:
            self._add_hidden(l, u, x, x.shape[0], w2, B.MQA_EPI_ADD)
            self._norm(x, out, packed)
        else:
            self._add_hidden(l, u, ws, x.shape[0], w2, B.MQA_EPI_STORE)
            B.mqa_stack_layernorm_packed(x, packed, out=out, parts=ws, S=w2 & 15)

    def _norm(self, x, out, packed):
        if packed is None:
            B.mqa_stack_layernorm(x, out=out)
        else:
            B.mqa_stack_layernorm_packed(x, packed, out=out)

    def _project_norm(self, mode, src, P, x, ws, out, packed):
        if packed is None:
            B.mqa_project_add_layernorm(mode, src, P, x, out=out, workspace=ws)
        else:
            B.mqa_stack_add_layernorm_packed(mode, src, P, x, packed, out=out, workspace=ws)

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

    def _workspace(self, plans, rows: int, kv_rows: int = 0) -> torch.Tensor:
        """Scratch memory for the calls of one pass over `rows` rows, one after another on its stream (a pass's own: calls on several
        streams do not share it)."""
        nbytes = self._parts.get(rows)         # (a decoding loop asks for the same rows again and again: 1.5 us of a step)
        if nbytes is None:
            sizes = [B.mqa_project_add_layernorm_workspace_bytes(B.MQA_PROJ_O, rows, self.d, self.h, self.v)]
            for ff in {w["W1"].shape[1] for w in self.layers}:
                sizes.append(B.mqa_project_add_layernorm_workspace_bytes(B.MQA_PROJ_LINEAR, rows, ff, 1, self.d))
            if rows == self.b:                 # (a step's attention)
                dt = B._cache_dtype(self.K[0])
                sizes.append(B.mqa_decode_workspace_bytes_default(self.b, self.h, self.cap, self.k, self.v, dt, self.multi_head))
            if len(self._parts) >= 16:
                self._parts.clear()
            nbytes = self._parts[rows] = max(sizes)
        parts = max(plan[1] & 15 for plan in plans)
        return torch.empty(max(nbytes, kv_rows, 16, 4 * parts * rows * self.d if parts > 1 else 0), dtype=torch.uint8, device=self.dev)

    # -- one decoding step for the whole stack: per layer 7 launches (fused q/K/V + append, attention (+ merge), output
    #    projection in parts, their sum added into x with the layernorm, W1 with relu, W2 in parts, the same)
    def step(self, tokens: torch.Tensor, t: int) -> torch.Tensor:
        x = self.embed(tokens, t)
        dec = B.mha_decode_step if self.multi_head else B.mqa_decode_step
        plans = self._plan(self.b)
        ws = self._workspace(plans, self.b)
        hx = B.mqa_stack_layernorm(x)
        rows = self._packed_rows(self.b, self.d) if any(plan[0] for plan in plans) else None
        for l, w in enumerate(self.layers):
            q = self._append_fused(l, hx)
            o = dec(q, self.K[l], self.V[l], self.lens[l], workspace=ws)
            packed = rows if plans[l][0] else None
            self._project_norm(B.MQA_PROJ_O, o, w["P_o"], x, ws, hx if packed is None else None, packed)
            self._feed_forward(l, plans[l], hx if packed is None else packed, x, ws, hx, None)
        return self._logits(hx)

    # -- a whole prompt at once (multi-query only): bulk append + fused causal attention per layer
    def prefill(self, prompts: torch.Tensor) -> torch.Tensor:
        """prompts [b,n] int32, caches empty.  Returns the logits of the last prompt position [b,vocab]."""
        if self.multi_head:
            raise NotImplementedError("prefill is built for the multi-query cache")
        b, n = prompts.shape
        rows = b * n
        positions = torch.arange(n, dtype=torch.int32, device=self.dev).repeat(b)
        x = B.mqa_stack_embed(prompts.reshape(-1).to(torch.int32).contiguous(), positions, self.E, self.pos)   # [b*n,d]
        plans = self._plan(rows)
        ws = self._workspace(plans, rows, B.mqa_project_kv_workspace_bytes(b, n, self.d, 1, self.k, self.v, B._cache_dtype(self.K[0])))
        hx = torch.empty_like(x)
        packed = self._packed_rows(rows, self.d) if any(plan[0] for plan in plans) else None
        end = len(self.layers) - 1
        B.mqa_stack_layernorm(x, out=hx)
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
                x = x.view(b, n, self.d)[:, n - 1].contiguous()
                rows, plans = b, self._plan(b)
                ws, hx = self._workspace(plans[end:], b), torch.empty_like(x)
                packed = self._packed_rows(b, self.d) if plans[end][0] else None
                B.mqa_stack_layernorm(x, out=hx)
            form_1, _, form_2 = plans[l]
            q = B.mqa_project_qkvo(B.MQA_PROJ_Q, hx, w["P_q"]).view(b, rows // b, self.h, self.k)
            o = B.mqa_prefill_attention(q, self.K[l], self.V[l], now, workspace=ws if l == end else None)
            self._project_norm(B.MQA_PROJ_O, o.view(rows, self.h, self.v), w["P_o"], x, ws, None if form_1 else hx, packed if form_1 else None)
            if l < end:
                self._feed_forward(l, plans[l], packed if form_1 else hx, x, ws, hx, None)
            else:                             # (logits() normalises)
                u = self._hidden(l, packed if form_1 else hx, rows, form_1, form_2)
                if form_2:
                    self._add_hidden(l, u, x, rows, form_2, B.MQA_EPI_ADD)
                else:
                    B.mqa_project_qkvo_ex(B.MQA_PROJ_LINEAR, u, w["W2"], out=x, epilogue=B.MQA_EPI_ADD)
        if now is not self.lens[-1]:      # the lengths advance in the arrays they are in: a caller may hold them
            torch._foreach_copy_(self.lens, self._lens_next)
        return self.logits(x)

    def greedy(self, logits: torch.Tensor) -> torch.Tensor:
        return B.mqa_stack_argmax(logits)
