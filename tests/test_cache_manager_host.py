"""The bookkeeping of the cache manager on the CPU: which token goes to which row, in which calls, and what is left after a call that
failed.  The two native calls are replaced by stand-ins on host memory: copies by memmove, the encoder by an arithmetic of its
own, row by row, in which every output depends on the row's K, V and previous reconstructions.  A plain loop over the tokens
of one sequence says what has to be where."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2501_19392_amd import binding as B
from paper_2501_19392_amd.cache import AquaKVCache

H, G = 2, 128
D = H * G
SINKS, RECENT = 3, 4


def make_layer(first=False):
    w = [None, None] if first else [torch.zeros(D, D), torch.zeros(D, 2 * D)]
    return B.Layer(H, G, torch.zeros(16, 2), torch.ones(D), torch.ones(D), torch.float32, w_k=w[0], w_v=w[1])


LAYER0, LAYER = make_layer(first=True), make_layer()


def rows(x, n, width, dtype):
    """n x width array over the memory of a tensor or an address"""
    if isinstance(x, torch.Tensor):
        x = x.data_ptr()
    size = n * width * np.dtype(dtype).itemsize
    return np.frombuffer((ctypes.c_char * size).from_address(x), dtype).reshape(n, width)


def arithmetic(K, V, Kp, Vp):
    """-> codes and scales of both, Khat, Vhat of rows of D floats"""
    Kh = np.round(K * 4) / 4 + (0 if Kp is None else 0.5 * Kp)
    Vh = np.round(V * 8) / 8 + 0.25 * Kh + (0 if Vp is None else 0.5 * Vp)
    out = []
    for x in (Kh, Vh):
        f = x.astype(np.float32)
        out += [f.view(np.uint8)[:, 5:5 + H * 32].copy(), f.view(np.int16)[:, 2:2 + H].copy()]
    return out, Kh.astype(np.float32), Vh.astype(np.float32)


class Calls:
    """Stand-ins for the native calls; the `fail_at`-th one raises."""
    def __init__(self, monkeypatch):
        self.n, self.fail_at, self.encoded = 0, None, []
        monkeypatch.setattr(B, "aquakv_copy_ranges", self.copy_ranges)
        monkeypatch.setattr(B, "aquakv_encode_layer", self.encode_layer)

    def count(self):
        self.n += 1
        if self.fail_at is not None and self.n > self.fail_at:
            raise B.AquaKVError(B.AQUAKV_EHIP)

    def copy_ranges(self, flat):
        self.count()
        flat = list(flat)
        for dst, src, size in zip(flat[::3], flat[1::3], flat[2::3]):
            ctypes.memmove(dst, src, size)

    def encode_layer(self, lay, N, K, V, Kp, Vp, kc, ks, vc, vs, Kh, Vh, ws):
        self.count()
        self.encoded.append(N)
        assert (Kp is None) == (Vp is None) == (lay.c.d_in_k == 0)
        assert ws.nbytes >= B.aquakv_workspace_bytes(lay, N)
        x = [None if p is None else rows(p, N, D, np.float32) for p in (K, V, Kp, Vp)]
        codes, Kr, Vr = arithmetic(*x)
        for dst, c, width, dt in zip((kc, ks, vc, vs), codes, (H * 32, H) * 2, (np.uint8, np.int16) * 2):
            rows(dst, N, width, dt)[:] = c
        rows(Kh, N, D, np.float32)[:] = Kr
        rows(Vh, N, D, np.float32)[:] = Vr


@pytest.fixture
def calls(monkeypatch):
    return Calls(monkeypatch)


def new_cache(layers, batch, max_tokens, **kw):
    cache = AquaKVCache(layers, max_tokens=max_tokens, sink_tokens=SINKS, buffer_tokens=RECENT, batch=batch, device="cpu", **kw)
    for t in [x for part in (cache.sink, cache.buf, cache.raw) for p in part if p is not None for x in p] + \
             [x for c in cache.codes if c is not None for p in c for x in p]:
        t.zero_()
    return cache


def stream(layers, batch, tokens, seed=0):
    gen = torch.Generator().manual_seed(seed)
    return [tuple(torch.randn(batch, tokens, H, G, generator=gen) for _ in range(2)) for _ in layers]


def content(cache):
    """What a cache holds, sequence by sequence and layer by layer: counts, sinks, compressed range, recent tokens."""
    out = []
    for b in range(cache.batch):
        ns, nc, nb = cache._ns[b], cache._nc[b], cache._nb[b]
        seq = [(ns, nc, nb)]
        for l in range(len(cache.layers)):
            held = cache.raw[l] if cache.raw[l] is not None else [t for p in cache.codes[l] for t in p]
            seq.append([t[b, :ns].numpy().copy() for t in cache.sink[l]] + [t[b, :nb].numpy().copy() for t in cache.buf[l]] +
                       [t[b * cache._C:b * cache._C + nc].numpy().copy() for t in held])
        out.append(seq)
    return out


def expected(layers, kv, lengths):
    out = []
    for b, n in enumerate(lengths):
        ns = min(n, SINKS)
        nc = (n - ns) // RECENT * RECENT
        seq, Kp, Vp = [(ns, nc, n - ns - nc)], None, None
        for lay, (K, V) in zip(layers, kv):
            Kc, Vc = (x[b, ns:ns + nc].reshape(nc, D).numpy() for x in (K, V))
            if lay is None:
                held, Kp, Vp = [x.reshape(nc, H, G) for x in (Kc, Vc)], Kc, Vc
            else:
                held, Kp, Vp = arithmetic(Kc, Vc, Kp, Vp)
                held = [h.reshape(nc, H, 32) if h.dtype == np.uint8 else h for h in held]
            seq.append([x[b, :ns].numpy() for x in (K, V)] + [x[b, ns + nc:n].numpy() for x in (K, V)] + held)
        out.append(seq)
    return out


def check(cache, kv, lengths):
    got, want = content(cache), expected(cache.layers, kv, lengths)
    for b, (g, w) in enumerate(zip(got, want, strict=True)):
        assert g[0] == w[0], b
        for l, (gl, wl) in enumerate(zip(g[1:], w[1:], strict=True)):
            for i, (x, y) in enumerate(zip(gl, wl, strict=True)):
                assert np.array_equal(x, y), (b, l, i)


STACKS = {"coded": [LAYER0, LAYER, LAYER], "raw first": [None, LAYER, LAYER], "raw inside": [LAYER0, None, LAYER]}


@pytest.mark.parametrize("stack", STACKS)
@pytest.mark.parametrize("batch", [1, 3])
def test_an_append_that_fails_can_be_made_again(calls, stack, batch):
    """Whichever of its native calls fails, an append leaves the counts and everything counted as they were, and the same
    append made again gives what it would have given at once."""
    layers, first = STACKS[stack], [9, 3 + 4 + 2, 2][:batch]
    then = [15, 2, 20][:batch]                     # tops up, flushes, goes on directly, ends in the buffer
    kv = stream(layers, batch, 40)

    def pieces(a, n):
        return [tuple(torch.stack([x[b, a[b]:a[b] + max(n)] for b in range(batch)]) for x in p) for p in kv]

    def filled():
        cache = new_cache(layers, batch, 40)
        cache.append(pieces([0] * batch, first), lengths=first)
        return cache

    cache = filled()
    calls.n = 0
    cache.append(pieces(first, then), lengths=then)
    total = calls.n
    check(cache, kv, [a + b for a, b in zip(first, then)])
    assert total > 4
    for k in range(total):
        cache = filled()
        before = content(cache)
        calls.n, calls.fail_at = 0, k
        with pytest.raises(B.AquaKVError):
            cache.append(pieces(first, then), lengths=then)
        calls.fail_at = None
        for x, y in zip(before, content(cache), strict=True):
            assert x[0] == y[0]
            assert all(np.array_equal(p, q) for r, s in zip(x[1:], y[1:]) for p, q in zip(r, s))
        cache.append(pieces(first, then), lengths=then)
        check(cache, kv, [a + b for a, b in zip(first, then)])


@pytest.mark.parametrize("stack", STACKS)
@pytest.mark.parametrize("batch", [1, 3])
def test_without_memory_for_scratch_a_prompt_goes_through_the_flush_buffers(calls, monkeypatch, stack, batch):
    layers, lengths = STACKS[stack], [40, 17, 5][:batch]
    kv = stream(layers, batch, 40, seed=1)
    cache = new_cache(layers, batch, 40)

    def no_memory(*a, **kw):
        raise torch.OutOfMemoryError("no memory")

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", no_memory)
        cache.append(kv, lengths=lengths)
    check(cache, kv, lengths)
    assert max(calls.encoded) <= batch * RECENT


@pytest.mark.parametrize("batch,lengths", [(1, None), (1, [19]), (3, [19, 4, 11]), (3, None)])
def test_tensors_with_more_or_fewer_rows_than_the_first_layers_keys(calls, batch, lengths):
    """Only the tokens that are taken have to be there: values and later layers may hold more rows (and sequences), or fewer."""
    layers, t = [LAYER0, LAYER, LAYER], 21
    full = stream(layers, batch + 1, 30, seed=2)
    taken = [t] * batch if lengths is None else lengths
    sizes = [(t, 30), (max(taken), 25), (22, max(taken))]
    kv = [tuple(x[:batch if (l, i) == (0, 0) else batch + i, :m].contiguous() for i, (x, m) in enumerate(zip(p, s)))
          for l, (p, s) in enumerate(zip(full, sizes))]
    cache = new_cache(layers, batch, 40)
    cache.append([tuple(x[0] for x in p) for p in kv] if batch == 1 else kv, lengths=lengths)
    check(cache, full, taken)
    with pytest.raises(RuntimeError):                    # a token that is not there
        short = [tuple(x[0, :max(taken) - 1] if batch == 1 else x[:, :max(taken) - 1] for x in p) for p in kv[1:]]
        new_cache(layers, batch, 40).append([tuple(x[0] if batch == 1 else x for x in kv[0])] + short, lengths=lengths)


@pytest.mark.parametrize("stack", STACKS)
@pytest.mark.parametrize("batch", [1, 3])
def test_replaced_tensors_are_the_ones_that_are_used(calls, monkeypatch, stack, batch):
    """Sinks, buffers, codes and 16-bit ranges replaced by copies between two calls: append and attend go by the copies."""
    layers, n = STACKS[stack], 34
    kv = stream(layers, batch, n, seed=3)
    cache, seen = new_cache(layers, batch, n), []
    monkeypatch.setattr(B, "aquakv_attend_cache", lambda entries, *a, **kw: seen.append([
        [getattr(e, f) for f in ("sink_k", "recent_v", "k_codes", "v_scales", "raw_k")] for e in entries]))
    q = [torch.zeros(batch, 2 * H, G) for _ in layers]

    def replace():
        for part in (cache.sink, cache.buf, cache.raw, cache.codes):
            for l, p in enumerate(part):
                if p is not None:
                    part[l] = tuple(tuple(t.clone() for t in x) if isinstance(x, tuple) else x.clone() for x in p)
                    for x in p:                              # the old ones are gone
                        for t in x if isinstance(x, tuple) else (x,):
                            t.fill_(77)

    def lies():
        return [[cache.sink[l][0].data_ptr(), cache.buf[l][1].data_ptr()] +
                ([None, None, cache.raw[l][0].data_ptr()] if lay is None else
                 [cache.codes[l][0][0].data_ptr(), cache.codes[l][1][1].data_ptr(), None]) for l, lay in enumerate(layers)]

    at = 0
    for step in (2, 3, 11, 1, 1, 16):
        cache.append([tuple(x[:, at:at + step] for x in p) for p in kv])
        at += step
        cache.attend([x[0] for x in q] if batch == 1 else q, 1.0)
        assert seen[-1] == lies()
        replace()
        cache.attend([x[0] for x in q] if batch == 1 else q, 1.0)
        assert seen[-1] == lies()
    assert at == n
    check(cache, kv, [n] * batch)


@pytest.mark.parametrize("batch", [1, 3])
def test_queries_that_are_copied_and_queries_that_are_refused(calls, monkeypatch, batch):
    layers, QH = [LAYER0, LAYER], 2 * H
    cache, seen = new_cache(layers, batch, 9), []
    monkeypatch.setattr(B, "aquakv_attend_cache", lambda entries, *a, **kw: seen.append(
        [rows(e.q, batch * QH, G, np.float32).copy() for e in entries]))
    cache.append(stream(layers, batch, 5))
    gen = torch.Generator().manual_seed(4)
    q = [torch.randn(batch + 2, QH, G, generator=gen) for _ in range(3)]

    def passed(make):
        cache.attend([make(x) for x in q], 1.0)
        for got, x in zip(seen[-1], q[:2], strict=True):
            assert np.array_equal(got, x[:batch].reshape(-1, G).numpy())

    passed(lambda x: x[0] if batch == 1 else x[:batch])                                  # one more than there are layers
    passed(lambda x: x)                                                                   # more sequences than the cache has
    passed(lambda x: x[:batch].transpose(1, 2).contiguous().transpose(1, 2))              # gaps
    passed(lambda x: torch.cat([torch.zeros(1), x[:batch].flatten()])[1:].view(batch, QH, G))        # not 16-byte aligned
    if batch > 1:
        passed(lambda x: x.double())
    else:
        with pytest.raises(ValueError):
            cache.attend([x[0].double() for x in q], 1.0)
    for bad in (lambda x: x[:, :, 1:], lambda x: x[:0]):
        with pytest.raises(ValueError):
            cache.attend([bad(x) for x in q], 1.0)
    with pytest.raises(ValueError):
        cache.attend([x[:batch] for x in q[:1]], 1.0)


@pytest.mark.parametrize("stack", STACKS)
@pytest.mark.parametrize("batch,lengths", [(1, [43]), (3, [43, 9, 30]), (3, [3, 43, 2]), (4, [11, 11, 11, 11])])
@pytest.mark.parametrize("limit", [1, RECENT, 3 * RECENT + 1, 7 * RECENT])
def test_prompts_longer_than_one_call_takes(calls, stack, batch, lengths, limit):
    """Chunks with one piece (written in place) and with several (gathered and scattered), sequences cut between chunks, scratch
    used again by the next chunk; with an empty cache and behind tokens that are already in the buffer."""
    layers, n = STACKS[stack], max(lengths) + 6
    kv = stream(layers, batch, n, seed=6)
    for head in (0, 5):                                  # 5: the sinks and two tokens in the buffer
        cache = new_cache(layers, batch, n)
        cache.kDirectTokens = limit
        calls.encoded.clear()
        if head:
            cache.append([tuple(x[:, :head] for x in p) for p in kv])
        cache.append([tuple(x[:, head:] for x in p) for p in kv], lengths=lengths)
        check(cache, kv, [head + m for m in lengths])
        flushed = sum(1 for m in lengths if head and SINKS < head < SINKS + RECENT <= head + m)
        assert max(calls.encoded, default=0) <= max(limit // RECENT * RECENT, RECENT, flushed * RECENT)


@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("what", ["dtype", "gaps between tokens", "gaps between heads", "heads by stride", "unaligned", "one head for all",
                                  "odd batch stride"])
def test_sources_that_have_to_be_copied(calls, what, batch):
    layers, n = [LAYER0, LAYER], 25
    kv = stream(layers, batch, n, seed=7)
    if what == "one head for all":
        kv = [tuple(x[:, :, :1].expand(batch, n, H, G).contiguous() for x in p) for p in kv]

    def source(x):
        if what == "dtype":
            return x.double()
        if what == "gaps between tokens":
            return torch.cat([x, x + 1], -2)[:, :, :H]
        if what == "gaps between heads":
            return torch.cat([x, x + 1], -1)[..., :G]
        if what == "heads by stride":
            return x.transpose(1, 2).contiguous().transpose(1, 2)
        if what == "unaligned":
            return torch.cat([torch.zeros(3), x.flatten()])[3:].view(x.shape)
        if what == "odd batch stride":
            return torch.cat([x.flatten(1), torch.zeros(batch, 1)], 1)[:, :-1].view(x.shape)
        return x[:, :, :1]

    for mix in (False, True):                            # every tensor, or the first layer's as they are
        cache = new_cache(layers, batch, n)
        src = [tuple(x if mix and l == 0 else source(x) for x in p) for l, p in enumerate(kv)]
        cache.append([tuple(x[0] for x in p) for p in src] if batch == 1 else src)
        check(cache, kv, [n] * batch)


@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("made", ["pairs", "tensors", "iterator"])
def test_sources_made_on_access(calls, made, batch):
    """Tensors that the given sequence makes when it is asked for them belong to nobody else: append holds them until all of its calls
    have been queued."""
    layers, n = [LAYER0, LAYER, LAYER], 25
    kv = stream(layers, batch, n, seed=8)
    new = lambda x: (x[0] if batch == 1 else x) * 1.0

    class Pair:
        def __init__(self, pair):
            self.pair = pair

        def __len__(self):
            return 2

        def __getitem__(self, i):
            return new(self.pair[i])

    class Made:
        def __len__(self):
            return len(kv)

        def __getitem__(self, l):
            return Pair(kv[l]) if made == "tensors" else tuple(new(x) for x in kv[l])

        if made == "iterator":
            def __iter__(self):
                return (tuple(new(x) for x in p) for p in kv)

    cache = new_cache(layers, batch, n)
    cache.append(Made())
    check(cache, kv, [n] * batch)
