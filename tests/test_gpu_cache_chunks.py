"""A prompt that the cache manager cuts into several calls per layer (kDirectTokens) against the same tokens given a buffer's worth at a
time, sequence by sequence: the same codes and scales, bit for bit, and the same 16-bit ranges."""
import pytest
import torch

from tests import parity_utils as U

pytestmark = pytest.mark.gpu
R, SINKS = 32, 4


@pytest.mark.parametrize("raw_layer", [None, 0, 1])
@pytest.mark.parametrize("rht_group", [None, 1024])
@pytest.mark.parametrize("lengths,limit", [([4 + 10 * R + 5], 3 * R), ([4 + 5 * R, 4 + 9 * R + 7, 30, 4 + R], 4 * R), ([600, 100, 601], 1)])
def test_chunks_give_the_codes_of_single_buffers(lengths, limit, rht_group, raw_layer):
    from paper_2501_19392_amd.cache import AquaKVCache
    print(f"case chunks lengths={lengths} limit={limit} group={rht_group} raw={raw_layer}", flush=True)
    L, H, D, NB, n = 3, 8, 1024, len(lengths), max(lengths)
    gen = torch.Generator().manual_seed(n + limit)
    layers, kv = [], []
    for l in range(L):
        w = {} if l == 0 else dict(w_k=U.random_weights(D, D, 31, 0.5), w_v=U.random_weights(D, 2 * D, 32, 0.5))
        layers.append(None if l == raw_layer else U.make_layers(H, "bf16", 256 if l == 0 else 16, layer_idx=l, rht_group=rht_group, **w)[1])
        kv.append(tuple(torch.randn(NB, n, H, 128, generator=gen).bfloat16().cuda() for _ in range(2)))
    cache = AquaKVCache(layers, max_tokens=n, sink_tokens=SINKS, buffer_tokens=R, batch=NB)
    cache.kDirectTokens = limit
    cache.append([(K[0], V[0]) if NB == 1 else (K, V) for K, V in kv], lengths=lengths)
    for b, m in enumerate(lengths):
        one = AquaKVCache(layers, max_tokens=n, sink_tokens=SINKS, buffer_tokens=R)
        for at in [0] + list(range(SINKS, m, R)):
            end = min(SINKS if at == 0 else at + R, m)
            one.append([(K[b, at:end], V[b, at:end]) for K, V in kv])
        torch.cuda.synchronize()
        c = one.n_compressed
        assert (cache._ns[b], cache._nc[b], cache._nb[b]) == (one.n_sink, c, one.n_buffered) and c == (m - SINKS) // R * R
        for l in range(L):
            held = [cache.raw[l], one.raw[l]] if layers[l] is None else [[t for p in x.codes[l] for t in p] for x in (cache, one)]
            for got, want in zip(*held):
                got, want = got[b * cache._C:b * cache._C + c], want[:c]
                assert torch.equal(got.contiguous().view(torch.uint8), want.contiguous().view(torch.uint8)), (b, l)
            for got, want in zip((*cache.sink[l], *cache.buf[l]), (*one.sink[l], *one.buf[l])):
                k = one.n_sink if got.shape[1] == SINKS else one.n_buffered
                assert torch.equal(got[b, :k], want[0, :k]), (b, l)
