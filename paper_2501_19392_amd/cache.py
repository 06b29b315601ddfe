"""Cache policy around the per-layer calls: attention sinks, recent-token buffer, flush and recovery, for a batch
of sequences.

AQUA-KV paper (arxiv 2501.19392), Sect. 3.3: the first few tokens ("attention sinks", 4 in the
experiments) stay in 16 bits; up to r = 128 recent tokens are kept uncompressed and, when that buffer
is full, quantized layer by layer from the first layer to the last; Alg. "Inference": to attend, the
compressed past is recovered one layer at a time, each layer from the previous layer's recovered past.

Sect. 4.1 (first-layer strategies): every layer brings its own grid (the paper's default quantizes the first layer,
which has no predictor, with the 4-bit grid), and a layer given as None is kept in 16 bits (its flushed tokens are
stored as they are and feed the next layer's predictors).

`attend` is the block call of Alg. "Inference" for one new token per sequence as far as the cache is concerned: per
layer the soft-max attention of that token's queries over everything cached, in one native call for all layers and
sequences (`aquakv_attend_cache`).

Batch.  Every sequence has its own sinks, buffer and compressed range (lengths may differ).  All sequences whose
buffer fills during one `append` are quantized together: ONE `aquakv_encode_layer` per layer (or one `aquakv_encode_layers`
for all, where no tokens have to be gathered) over (number of full buffers) x r tokens; whole buffers' worth of a prompt go from the caller's tensors to the compressed
range directly.  Codes of a sequence are contiguous in its own range of the code tensors; `attend` recovers a layer of
all sequences at once, from codes that are first put one behind the other in a staging range unless they already are
(codes are an eighth of the bytes the recovery moves).

This class is bookkeeping only: every number is produced by the C-ABI calls (`aquakv_encode_layer`,
`aquakv_decode_layer`, the attention calls above); torch tensors are the device memory they work on.
"""
from __future__ import annotations

from typing import Iterator, List, Optional, Sequence, Tuple

import torch

from . import binding as B


class AquaKVCache:
    kDirectTokens = 32768          # tokens quantized per call when a prompt goes straight to the compressed range

    def __init__(self, layers: Sequence[B.Layer], max_tokens: int, sink_tokens: int = 4, buffer_tokens: int = 128,
                 device="cuda", batch: int = 1):
        """max_tokens: per sequence.  With batch == 1 the calls take and return tensors without the batch dimension."""
        if buffer_tokens < 1 or sink_tokens < 0 or batch < 1:
            raise ValueError("buffer_tokens >= 1, sink_tokens >= 0 and batch >= 1")
        self.layers = list(layers)
        self.sink_tokens, self.buffer_tokens, self.max_tokens, self.batch = sink_tokens, buffer_tokens, max_tokens, batch
        lay0 = next(l for l in self.layers if l is not None)
        H, g, dt = lay0.kv_heads, lay0.head_dim, lay0.dtype
        self._H, self._g, self._dt = H, g, dt
        L, S, R, buf = len(self.layers), max(sink_tokens, 1), batch * buffer_tokens, buffer_tokens
        cap = max(max_tokens - sink_tokens, 0) // buffer_tokens * buffer_tokens      # the compressed range grows by whole buffers
        self.capacity = cap
        C = max(cap, 1)
        self._C = C
        # A cache is made per request, so what it costs counts: tensors of one shape are slices of one allocation.
        raws = lambda n, *shape: torch.empty(n, *shape, H, g, dtype=dt, device=device).unbind(0)
        pairs = lambda ts: list(zip(ts[::2], ts[1::2]))
        self._like = torch.empty(0, dtype=dt, device=device)
        self._row_bytes = H * g * self._like.element_size()                          # one token's keys (or values)
        self.sink = pairs(raws(2 * L, batch, S))
        self.buf = pairs(raws(2 * L, batch, buf))
        # sequence b owns tokens [b * C, (b + 1) * C) of the code tensors (and of the 16-bit tensors of a layer given as None)
        self.codes = self._alloc_codes(batch * C, device)
        kept = sum(l is None for l in self.layers)
        raw = iter(pairs(raws(2 * kept, batch * C)) if kept else ())
        self.raw = [next(raw) if l is None else None for l in self.layers]
        # flush: reconstructions of the flushed tokens, two ping-pong pairs (layer l - 1 feeds layer l); with several
        # sequences also the gathered buffers and the codes before they are scattered to their sequences
        self._flush_hat = pairs(raws(4, R))
        self._flush_ws = self._alloc_workspace(R, device)
        self._flush_in = pairs(raws(4, R)) if batch > 1 else None
        self._flush_codes = self._alloc_codes(R, device) if batch > 1 else [None] * L
        # recovery: [sinks | compressed | buffer] of one layer and sequence (sweep), or the compressed ranges of all
        # sequences (attend, which puts their codes one behind the other first): two ping-pong pairs
        self._view = pairs(raws(4, max(max_tokens, batch * C)))
        self._view_ws = self._alloc_workspace(batch * C, device)
        self._staged = self._alloc_codes(batch * C, device) if batch > 1 else [None] * L
        self._ns, self._nc, self._nb = [0] * batch, [0] * batch, [0] * batch
        # all layers of a flush, or of a prompt, in one native call (aquakv_encode_layers) where their tokens lie one behind the other;
        # fp32 layers, and predictors of other widths, layer by layer
        D = H * g
        self._one_call = dt == torch.bfloat16 and all(l is None or (l.kv_heads * l.head_dim == D and l.c.d_in_k in (0, D) and
                                                                    l.c.d_in_v in (0, 2 * D)) for l in self.layers)
        self._attend = None                 # buffers of attend(), sized on first use (they depend on the query heads)
        self._device = device

    def _alloc_codes(self, tokens: int, device) -> list:
        """((k codes, k scales), (v codes, v scales)) per layer, None where the layer is; layers of one format share two
        allocations."""
        kinds = {}
        for l, lay in enumerate(self.layers):
            if lay is not None:
                kinds.setdefault((lay.n_codewords, lay.rtn_bits, lay.rht_group), []).append(l)
        out = [None] * len(self.layers)
        for members in kinds.values():
            codes, scales = self.layers[members[0]].alloc_codes(2 * len(members) * tokens, device)
            both = list(zip(codes.split(tokens), scales.split(tokens)))
            for i, l in enumerate(members):
                out[l] = (both[2 * i], both[2 * i + 1])
        return out

    def _alloc_workspace(self, tokens: int, device) -> torch.Tensor:
        """For encoding and decoding `tokens` tokens at any layer; with groups across the heads also room for the predictions
        of a short range, which is then encoded in one piece."""
        d = self._H * self._g
        need = {(l.n_codewords, l.rtn_bits, l.rht_group, l.c.d_in_k, l.c.d_in_v): l for l in self.layers if l is not None}
        size = max(B.aquakv_workspace_bytes(l, tokens) + (min(tokens, 4096) * d * 4 if l.rht_group == d and self._H > 1 else 0) for l in need.values())
        return torch.empty(max(size, 16), dtype=torch.uint8, device=device)

    # ------------------------------------------------------------------ counts
    def _count(self, per_seq: List[int]):
        return per_seq[0] if self.batch == 1 else tuple(per_seq)

    @property
    def n_sink(self):
        return self._count(self._ns)

    @property
    def n_compressed(self):
        return self._count(self._nc)

    @property
    def n_buffered(self):
        return self._count(self._nb)

    @property
    def n_tokens(self):
        return self._count([s + c + b for s, c, b in zip(self._ns, self._nc, self._nb)])

    # ------------------------------------------------------------------ addresses
    # Taken from the tensors on every call: sink, buf, codes and raw may be replaced by others of the same layout (a cache
    # that is read back, say), and none of their addresses is kept.
    @staticmethod
    def _addresses(pairs) -> List[int]:
        return [t.data_ptr() for pair in pairs for t in pair]

    def _codes_at(self, l: int) -> List[Tuple[int, int]]:
        """(address, bytes per token) of the four code tensors of layer l"""
        return [(t.data_ptr(), t.stride(0) * t.element_size()) for pair in self.codes[l] for t in pair]

    # ------------------------------------------------------------------ append / flush
    def append(self, kv: Sequence[Tuple[torch.Tensor, torch.Tensor]], lengths: Optional[Sequence[int]] = None) -> None:
        """kv[l] = (K, V) of the new tokens at layer l in the storage dtype: [t, kv_heads, head_dim] for a single
        sequence, [batch, t, kv_heads, head_dim] otherwise; `lengths[b]` <= t tokens of sequence b are taken
        (default: all t).  Tensors of another dtype or device, and such with gaps, are copied.  If the call fails, the cache
        is what it was."""
        if len(kv) != len(self.layers):
            raise ValueError("one (K, V) pair per layer")
        first = kv[0][0]
        single = first.dim() == 3
        if single and self.batch != 1:
            raise ValueError("a batched cache takes [batch, t, kv_heads, head_dim]")
        t = first.shape[0] if single else first.shape[1]
        n = [t] * self.batch if lengths is None else [int(x) for x in lengths]
        if len(n) != self.batch or (not single and first.shape[0] != self.batch) or any(x < 0 or x > t for x in n):
            raise ValueError("one length per sequence, each at most the tokens given")
        if any(self._ns[b] + self._nc[b] + self._nb[b] + n[b] > self.max_tokens for b in range(self.batch)):
            raise ValueError("cache is full")
        # the sources: (address, bytes from sequence to sequence) per layer, keys then values.  `kept` holds the tensors behind the
        # addresses until all calls have been queued: copies made here, and what `kv` may have made when it was asked.
        most = max(n)
        like, es = self._like, self._like.element_size()
        dtype, device, kept, src = like.dtype, like.device, [], []
        usual = (t, self._H, self._g) if single else (self.batch, t, self._H, self._g)
        per_seq = 0 if single else t * self._row_bytes
        # A generated token brings two tensors per layer, and looking at them is most of what it costs on the host: those that are
        # as they should be are recognised in one go (8 layers: 29 -> 21 us a token).
        for pair in kv:
            for x in pair:
                if x.shape == usual and x.dtype is dtype and x.device == device and x.is_contiguous():
                    at = x.data_ptr()
                    if not at & 15:
                        kept.append(x)
                        src.append((at, per_seq))
                        continue
                x = self._rows(x, t, most)
                kept.append(x)
                src.append((x.data_ptr(), x.stride(0) * es if x.dim() == 4 else 0))
        # Per sequence: sinks first, then what tops up a buffer that already holds tokens, then whole buffers' worth of
        # tokens, which need no stop in the buffer, then the rest into the (by now empty) buffer.  The tokens land where
        # filling and flushing buffer after buffer would put them; what changes is that a prompt is quantized in one call
        # per layer over all its whole buffers instead of one call per 128 tokens (2436 tokens, 8 layers: 25.2 ms as 19
        # flushes per layer).
        # The counts move once everything has been queued: until then the tokens go to rows that are not counted (but for the
        # very last copy), so an append that fails can be made again.
        ns, nc, nb = list(self._ns), list(self._nc), list(self._nb)
        now, later, full, direct = [], [], [], []
        buf_at, sink_at = self._addresses(self.buf), None
        for b in range(self.batch):
            pos, left = 0, n[b]
            take = min(self.sink_tokens - ns[b], left)
            if take > 0:
                sink_at = sink_at or self._addresses(self.sink)
                self._store(now, sink_at, max(self.sink_tokens, 1), ns[b], src, b, pos, take)
                ns[b] += take
                pos, left = pos + take, left - take
            r, dst = self.buffer_tokens, now
            if nb[b] and left:
                take = min(r - nb[b], left)
                self._store(now, buf_at, r, nb[b], src, b, pos, take)
                nb[b] += take
                pos, left = pos + take, left - take
                if nb[b] == r:
                    full.append((b, nc[b]))
                    nc[b] += r
                    nb[b] = 0
                    dst = later                      # the buffer is free again once it has been flushed
            whole = left // r * r
            if whole:
                direct.append((b, pos, nc[b], whole))
                nc[b] += whole
                pos, left = pos + whole, left - whole
            if left:
                self._store(dst, buf_at, r, 0, src, b, pos, left)
                nb[b] = left
        plan = self._plan_direct(direct) if direct else None       # allocates, hence ahead of the first launch
        if now:
            B.aquakv_copy_ranges(now)
        if full:
            self._flush(full)
        if plan is not None:
            self._encode_direct(src, plan)
        if later:
            B.aquakv_copy_ranges(later)
        self._ns, self._nc, self._nb = ns, nc, nb

    def _rows(self, x: torch.Tensor, t: int, most: int) -> torch.Tensor:
        """x in the storage dtype on the cache's device, every sequence's tokens one contiguous block: as it is
        ([t, kv_heads, head_dim], [batch, t, kv_heads, head_dim]) or a copy.  `most` tokens are taken at most: a tensor may
        hold another number of rows (or sequences) than the first layer's keys, as long as those are among them."""
        H, g, like = self._H, self._g, self._like
        one = x.dim() == 3
        if x.shape != ((t, H, g) if one else (self.batch, t, H, g)):
            x, t = x[:most] if one else x[:self.batch, :most], most
        if x.dtype != like.dtype or x.device != like.device or x.shape != ((t, H, g) if one else (self.batch, t, H, g)):
            x = x.to(device=like.device, dtype=self._dt).expand(self.batch, t, H, g)
            one = False
        if not (x.is_contiguous() and x.data_ptr() & 15 == 0):
            st = x.stride() if not one else (0, *x.stride())
            if st[3] != 1 or st[2] != g or (t > 1 and st[1] != H * g) or (x.data_ptr() | st[0] * x.element_size()) & 15:
                x = x.clone(memory_format=torch.contiguous_format)
        return x

    def _store(self, out: List[int], dst: List[int], rows: int, at: int, src, b: int, pos: int, take: int) -> None:
        """Adds the copies of tokens pos ... pos + take - 1 of sequence b, every layer, to row `at` of the sequence's `rows`
        rows of dst."""
        row = self._row_bytes
        to, pos, size = (b * rows + at) * row, pos * row, take * row
        for d, (x, seq) in zip(dst, src):
            out += (d + to, x + b * seq + pos, size)

    def _plan_direct(self, pieces: List[Tuple[int, int, int, int]]) -> tuple:
        """pieces: (sequence, first token in the source, first row of the sequence's compressed range, tokens): whole buffers'
        worth of tokens that go from the caller's tensors to the compressed range.  -> (chunks of pieces, one
        aquakv_encode_layer call per layer each, and the addresses of their scratch: reconstructions, gathered tokens, codes
        per layer before they are scattered).  A chunk has at most kDirectTokens tokens, which bounds the scratch; where not
        even that can be allocated, the buffers of the flush serve, with fewer tokens per chunk."""
        r, row = self.buffer_tokens, self._row_bytes

        def cut(limit):
            chunks, room = [[]], limit
            for b, pos, at, left in pieces:
                while left:
                    if not room:
                        chunks.append([])
                        room = limit
                    take = min(left, room)
                    chunks[-1].append((b, pos, b * self._C + at, take))
                    pos, at, left, room = pos + take, at + take, left - take, room - take
            return chunks

        chunks = cut(max(self.kDirectTokens // r, 1) * r)
        biggest = max(sum(p[3] for p in c) for c in chunks)
        gather = any(len(c) > 1 for c in chunks)
        # rows of codes and scales, the widest layer's
        coded = [self._codes_at(l) for l, c in enumerate(self.codes) if c is not None] if gather else []
        width = [max(p[i][1] for p in coded) for i in range(4)] if gather else []
        sizes = [biggest * row] * (8 if gather else 4) + [(biggest * w + 15) // 16 * 16 for w in width]
        try:
            scratch = torch.empty(sum(sizes), dtype=torch.uint8, device=self._like.device)
        except torch.OutOfMemoryError:
            pair = lambda ts: [tuple(t.data_ptr() for t in p) for p in ts]
            own = [None if c is None else self._addresses(c) for c in self._flush_codes]
            return cut(self.batch * r), pair(self._flush_hat), pair(self._flush_in or []), own, None
        at = [scratch.data_ptr()]
        for size in sizes:
            at.append(at[-1] + size)
        return chunks, [at[0:2], at[2:4]], [at[4:6], at[6:8]], [at[8:12]] * len(self.layers), scratch

    def _encode_direct(self, src, plan: tuple) -> None:
        """The chunks of _plan_direct, each from the first layer to the last."""
        row = self._row_bytes
        chunks, hat, stage, staged, _ = plan                           # layer l - 1 feeds layer l: two pairs of hat and stage
        for c in chunks:
            N = sum(p[3] for p in c)
            if self._one_call and len(c) == 1:
                b, pos, at, _ = c[0]
                Xs = [x + b * seq + pos * row for x, seq in src]
                self._encode_layers(N, Xs, [None if lay is None else [p + at * size for p, size in self._codes_at(l)]
                                            for l, lay in enumerate(self.layers)], hat, self._view_ws, [(at, N)])
                continue
            Kp = Vp = None
            for l, lay in enumerate(self.layers):
                Xs = [x + c[0][0] * seq + c[0][1] * row for x, seq in src[2 * l:2 * l + 2]]
                if len(c) > 1:
                    jobs, to = [], 0
                    for b, pos, _, m in c:
                        for X, (x, seq) in zip(stage[l & 1], src[2 * l:2 * l + 2]):
                            jobs += (X + to * row, x + b * seq + pos * row, m * row)
                        to += m
                    B.aquakv_copy_ranges(jobs)
                    Xs = stage[l & 1]
                if lay is None:                                        # kept in 16 bits
                    self._scatter([(t.data_ptr(), row) for t in self.raw[l]], Xs, [p[2:] for p in c])
                    Kp, Vp = Xs
                    continue
                Kh, Vh = hat[l & 1]
                stores = self._codes_at(l)
                out = [p + c[0][2] * size for p, size in stores] if len(c) == 1 else staged[l]
                B.aquakv_encode_layer(lay, N, *Xs, Kp, Vp, *out, Kh, Vh, self._view_ws)
                if len(c) > 1:
                    self._scatter(stores, out, [p[2:] for p in c])
                Kp, Vp = Kh, Vh

    def _encode_layers(self, N: int, Xs: List[int], outs: list, hat, ws, parts: List[Tuple[int, int]]) -> None:
        """N tokens whose K and V lie at addresses Xs[2 l], Xs[2 l + 1], one behind the other: codes and scales to outs[l], the rows of
        a layer kept in 16 bits to its ranges `parts`."""
        B.aquakv_encode_layers([(lay, *Xs[2 * l:2 * l + 2], *(outs[l] or (0, 0, 0, 0))) for l, lay in enumerate(self.layers)], N,
                               [x for pair in hat for x in pair], ws)
        jobs: List[int] = []
        for l, lay in enumerate(self.layers):
            if lay is None:
                self._scatter([(t.data_ptr(), self._row_bytes) for t in self.raw[l]], Xs[2 * l:2 * l + 2], parts, jobs)
        if jobs:
            B.aquakv_copy_ranges(jobs)

    @staticmethod
    def _scatter(stores, sources, parts: List[Tuple[int, int]], jobs: Optional[List[int]] = None) -> None:
        """The rows at address sources[k], part after part, to rows at ... of stores[k] = (address, bytes per row); added to
        `jobs`, or copied at once without."""
        own = [] if jobs is None else jobs
        for (to, row), frm in zip(stores, sources):
            for at, m in parts:
                own += (to + at * row, frm, m * row)
                frm += m * row
        if jobs is None:
            B.aquakv_copy_ranges(own)

    def _flush(self, full: List[Tuple[int, int]]) -> None:
        """The full buffers of the sequences `full` = (sequence, tokens in its compressed range) are quantized together from
        the first layer to the last; each sequence's codes land behind its own compressed range."""
        r, C, n = self.buffer_tokens, self._C, len(full)
        row = self._row_bytes
        single = self.batch == 1
        whole = n == self.batch                              # the buffers of all sequences are one contiguous tensor
        parts = [(b * C + at, r) for b, at in full]
        scatter: List[int] = []
        if whole and self._one_call:
            outs = [None if lay is None else [p + full[0][1] * size for p, size in self._codes_at(l)] if single
                    else self._addresses(self._flush_codes[l]) for l, lay in enumerate(self.layers)]
            self._encode_layers(n * r, self._addresses(self.buf), outs, self._flush_hat, self._flush_ws, parts)
            for l, lay in enumerate(self.layers):
                if not single and lay is not None:
                    self._scatter(self._codes_at(l), outs[l], parts, scatter)
            if scatter:                                      # the codes of all layers in one go
                B.aquakv_copy_ranges(scatter)
            return
        Kp = Vp = None
        for l, lay in enumerate(self.layers):
            if whole:
                Xk, Xv = self.buf[l]
            else:
                Xk, Xv = self._flush_in[l & 1]
                jobs: List[int] = []
                for X, x in ((Xk, self.buf[l][0]), (Xv, self.buf[l][1])):
                    for i, (b, _) in enumerate(full):
                        jobs += (X.data_ptr() + i * r * row, x.data_ptr() + b * r * row, r * row)
                B.aquakv_copy_ranges(jobs)
            if lay is None:                                  # kept in 16 bits: stored as is, feeds the next layer exactly
                self._scatter([(t.data_ptr(), row) for t in self.raw[l]], (Xk.data_ptr(), Xv.data_ptr()), parts)
                Kp, Vp = Xk, Xv
                continue
            Kh, Vh = (t.data_ptr() for t in self._flush_hat[l & 1])
            if single:
                out = [p + full[0][1] * size for p, size in self._codes_at(l)]
            else:
                out = self._addresses(self._flush_codes[l])
            B.aquakv_encode_layer(lay, n * r, Xk, Xv, Kp, Vp, *out, Kh, Vh, self._flush_ws)
            if not single:
                self._scatter(self._codes_at(l), out, parts, scatter)
            Kp, Vp = Kh, Vh
        if scatter:
            B.aquakv_copy_ranges(scatter)

    # ------------------------------------------------------------------ recovery of one sequence
    def sweep(self, seq: int = 0) -> Iterator[Tuple[int, torch.Tensor, torch.Tensor]]:
        """Yield (layer, K, V) of sequence `seq` for every layer in order, K and V being [n_tokens, kv_heads,
        head_dim]: sinks, the recovered compressed past, the buffered tokens.  The tensors are views of two
        ping-pong buffers: layer l's are valid until layer l + 2 is produced."""
        s, c, b = self._ns[seq], self._nc[seq], self._nb[seq]
        at = seq * self._C
        Kp = Vp = None
        for l, lay in enumerate(self.layers):
            K, V = self._view[l & 1]
            if s:
                K[:s].copy_(self.sink[l][0][seq, :s]); V[:s].copy_(self.sink[l][1][seq, :s])
            if c and lay is None:
                K[s:s + c].copy_(self.raw[l][0][at:at + c]); V[s:s + c].copy_(self.raw[l][1][at:at + c])
                Kp, Vp = K[s:s + c], V[s:s + c]
            elif c:
                (kc, ks), (vc, vs) = self.codes[l]
                B.aquakv_decode_layer(lay, c, kc[at:at + c], ks[at:at + c], vc[at:at + c], vs[at:at + c], Kp, Vp,
                                      K[s:s + c], V[s:s + c], self._view_ws)
                Kp, Vp = K[s:s + c], V[s:s + c]
            if b:
                K[s + c:s + c + b].copy_(self.buf[l][0][seq, :b]); V[s + c:s + c + b].copy_(self.buf[l][1][seq, :b])
            yield l, K[:s + c + b], V[:s + c + b]

    # ------------------------------------------------------------------ attention of one new token per sequence
    def attend(self, queries: Sequence[torch.Tensor], score_scale: float, rope=None) -> List[torch.Tensor]:
        """queries[l]: the new token's queries at layer l in the storage dtype, [q_heads, head_dim] for a single
        sequence, [batch, q_heads, head_dim] otherwise.  Queries on another device and such with gaps are copied; those of
        another dtype are converted for a batch and refused for a single sequence.  Returns one fp32 tensor of the same shape per layer:
        softmax(score_scale * q K^T) V over sinks, compressed past and buffer of the query's own sequence.
        One sweep over the layers for all sequences (aquakv_attend_cache); the recovered tensors of layer l feed
        layer l + 1 as in `sweep`.
        rope = (cos, sin), device fp32 [>= n_tokens, head_dim / 2]: the cache holds keys from before the rotary
        embedding (Sect. 3.3, the paper's default); the key of token t of a sequence is rotated by row t on the fly,
        the queries are taken as already rotated, and what is recovered for the next layer stays unrotated."""
        if any(s + c + b == 0 for s, c, b in zip(self._ns, self._nc, self._nb)):
            raise ValueError("nothing cached")
        single = queries[0].dim() == 2
        if single and self.batch != 1:
            raise ValueError("a batched cache takes [batch, q_heads, head_dim]")
        QH = queries[0].shape[-2]
        held = self._held()
        if self._attend is None or self._attend["shape"].q_heads != QH or self._attend["held"] != held:
            self._attend = dict(self._attend_state(QH), held=held)
        A = self._attend
        shape = (QH, self._g) if single else (self.batch, QH, self._g)
        if len(queries) < len(self.layers):
            raise ValueError("queries of every layer are needed")
        kept = [self._query(q, shape) for q in queries[:len(self.layers)]]      # copies must live until the call has been queued
        for entry, q in zip(A["layers"], kept):
            entry.q = q.data_ptr()
        cos, sin = rope if rope is not None else (None, None)
        B.aquakv_attend_cache(A["layers"], A["shape"], self._ns, self._nc, self._nb, score_scale, A["hat"], A["ws"], cos, sin)
        return [o[0] if single else o for o in A["out"]]

    def _query(self, q: torch.Tensor, shape: Tuple[int, ...]) -> torch.Tensor:
        like = self._like
        if len(shape) == 3 and q.dim() == 3 and q.shape[0] > shape[0]:
            q = q[:shape[0]]                                 # more sequences than the cache has
        if q.shape != shape or (q.dtype != like.dtype and self.batch == 1):
            raise ValueError(f"queries must be {list(shape)}, {self._dt}")
        if q.dtype != like.dtype or q.device != like.device:
            q = q.to(device=like.device, dtype=like.dtype)
        return q if q.is_contiguous() and q.data_ptr() & 15 == 0 else q.clone(memory_format=torch.contiguous_format)

    def _held(self) -> tuple:
        """What attend() passes on by address: the layers' descriptors and where everything that is cached lies."""
        return ([None if lay is None else lay.c for lay in self.layers],
                self._addresses(self.sink), self._addresses(self.buf), self._addresses(p for p in self.raw if p is not None),
                [t.data_ptr() for c in self.codes if c is not None for pair in c for t in pair])

    def _attend_state(self, q_heads: int) -> dict:
        """What attend() passes on every call for this number of query heads."""
        out = [torch.empty(self.batch, q_heads, self._g, dtype=torch.float32, device=self._device) for _ in self.layers]
        entries = []
        for l, lay in enumerate(self.layers):
            fields = dict(sink_k=self.sink[l][0], sink_v=self.sink[l][1], recent_k=self.buf[l][0], recent_v=self.buf[l][1], out=out[l])
            if lay is None:
                fields.update(raw_k=self.raw[l][0], raw_v=self.raw[l][1])
            else:
                names = ("k_codes", "k_scales", "v_codes", "v_scales")
                fields.update(zip(names, (t for pair in self.codes[l] for t in pair)))
                if self._staged[l] is not None:
                    fields.update(zip(("staged_" + n for n in names), (t for pair in self._staged[l] for t in pair)))
            entries.append((lay, fields))
        layers = B.cache_layers(entries)
        shape = B.aquakv_cache_shape(B._dtype_code(self._dt), self._H, q_heads, self.batch, max(self.sink_tokens, 1),
                                     self.buffer_tokens, self._C)
        ws = torch.empty(B.aquakv_attend_cache_workspace_bytes(layers, shape), dtype=torch.uint8, device=self._device)
        return dict(layers=layers, shape=shape, out=out, ws=ws, hat=[t for pair in self._view for t in pair])

    def stored_bytes(self) -> int:
        """Bytes the cache content occupies (all layers, all sequences): 16-bit sinks and buffer, packed codes and
        fp16 scales."""
        lay0 = next(l for l in self.layers if l is not None)
        per_tok = lay0.d * self.sink[0][0].element_size() * 2
        total = (sum(self._ns) + sum(self._nb)) * per_tok * len(self.layers)
        n_compressed = sum(self._nc)
        for lay in self.layers:
            if lay is None:
                total += n_compressed * per_tok
                continue
            groups = lay.d // lay.rht_group
            total += 2 * n_compressed * (lay.kv_heads * lay.code_bytes_per_group + 2 * groups * lay.scale_words_per_group)
        return total
