"""aquakv_attend_cache through the cache manager: attention of one new token per sequence against a plain soft-max in fp64 over the
tensors that the manager's own sweep recovers.  Lengths at the edges of the 64-token pieces, sequences with and without
compressed tokens side by side, ranges that need not be gathered, more sequences than one launch takes, layers in the storage
dtype, every number of query heads per kv head, and a workspace that holds one layer's partial results."""
import pytest
import torch

from paper_2501_19392_amd import synth
from tests import parity_utils as U

pytestmark = pytest.mark.gpu


def plain_attention(q, K, V, scale, rope):
    """q [QH, 128], K, V [n, H, 128] -> [QH, 128] in fp64"""
    q, K, V = q.double(), K.double(), V.double()
    if rope is not None:
        c, s = (t[:K.shape[0], None].double() for t in rope)
        lo, hi = K[..., :64], K[..., 64:]
        K = torch.cat([lo * c - hi * s, hi * c + lo * s], -1)
    rep = q.shape[0] // K.shape[1]
    K, V = K.repeat_interleave(rep, 1), V.repeat_interleave(rep, 1)
    p = torch.softmax((K * q[None]).sum(-1) * scale, 0)
    return (p[..., None] * V).sum(0)


@pytest.mark.parametrize("dtype,H,QH,sinks,recent,lengths,raw_layers,rope", [
    ("bf16", 8, 32, 4, 16, [63, 64, 65, 5], (), True), ("bf16", 8, 8, 4, 16, [128, 129, 1, 191], (1,), False),
    ("fp32", 2, 16, 0, 8, [64, 72, 9], (0,), True), ("bf16", 2, 2, 3, 100, [100, 320, 17], (), True),
    ("bf16", 1, 3, 2, 6, [8 + i % 25 for i in range(70)], (), True), ("bf16", 4, 20, 4, 16, [260], (2,), True),
    ("bf16", 8, 64, 4, 32, [4 + 64 + 7] * 3, (), False), ("fp32", 1, 8, 4, 8, [3], (), False),
    ("bf16", 2, 34, 4, 16, [150, 20], (), True)])                  # 17 query heads per kv head: in passes of 8, 8 and 1
def test_attend_over_ragged_caches(dtype, H, QH, sinks, recent, lengths, raw_layers, rope):
    from paper_2501_19392_amd.cache import AquaKVCache
    print(f"case attend cache dtype={dtype} H={H} QH={QH} sinks={sinks} recent={recent} lengths={lengths[:8]} raw={raw_layers} "
          f"rope={rope}", flush=True)
    L, NB, n, D = 3, len(lengths), max(lengths), H * 128
    sd = synth.torch_dtype(dtype)
    gen = torch.Generator().manual_seed(n + QH)
    layers, kv, qs = [], [], []
    for l in range(L):
        w = [None, None]
        if l > 0:
            w = [0.3 * torch.randn(D, d, generator=gen) / d ** 0.5 for d in (D, 2 * D)]
        lay = U.make_layers(H, dtype, 16, layer_idx=l, w_k=w[0], w_v=w[1])[1]
        layers.append(None if l in raw_layers else lay)
        kv.append(tuple(torch.randn(NB, n, H, 128, generator=gen).to(sd).cuda() for _ in range(2)))
        qs.append((2.0 * torch.randn(NB, QH, 128, generator=gen)).to(sd).cuda())
    tables = tuple(f(torch.rand(n, 64, generator=gen) * 6).float().cuda() for f in (torch.cos, torch.sin)) if rope else None
    cache = AquaKVCache(layers, max_tokens=n, sink_tokens=sinks, buffer_tokens=recent, batch=NB)
    single = NB == 1
    cache.append([(K[0], V[0]) if single else (K, V) for K, V in kv], lengths=None if single else lengths)
    scale = 128 ** -0.5
    got = [o.clone().view(NB, QH, 128) for o in cache.attend([q[0] if single else q for q in qs], scale, tables)]
    # the same with room for the partial results of one layer only
    whole = cache._attend["ws"]
    per_layer = (sum(-(-t // 64) for t in lengths) * QH * 130 * 4 + 255) // 256 * 256
    codec = max([lay.alloc_workspace(NB * cache._C).numel() for lay in layers if lay is not None])
    cache._attend["ws"] = torch.empty((codec + 255) // 256 * 256 + per_layer, dtype=torch.uint8, device="cuda")
    again = [o.clone().view(NB, QH, 128) for o in cache.attend([q[0] if single else q for q in qs], scale, tables)]
    cache._attend["ws"] = whole
    for l in range(L):
        assert torch.equal(got[l], again[l])
    for b in range(NB):
        for l, K, V in cache.sweep(b):
            want = plain_attention(qs[l][b], K, V, scale, tables)
            err = (got[l][b].double() - want).abs().max() / V.double().square().mean().sqrt()
            assert err < 1e-5, (b, l, float(err))


@pytest.mark.parametrize("n", [65, 130])
@pytest.mark.parametrize("what", ["values of the last token", "scores of a piece"])
def test_infinities_stay_where_they_are(n, what):
    """Tokens behind the end of a sequence and pieces whose scores are all -inf add nothing, not 0 x infinity."""
    from paper_2501_19392_amd.cache import AquaKVCache
    print(f"case attend infinities n={n} {what}", flush=True)
    lay = U.make_layers(1, "bf16", 16)[1]
    cache = AquaKVCache([lay], max_tokens=n, sink_tokens=0, buffer_tokens=256)          # everything in the buffer
    gen = torch.Generator().manual_seed(n)
    K, V = (torch.randn(n, 1, 128, generator=gen).bfloat16().cuda() for _ in range(2))
    q = torch.randn(1, 128, generator=gen).bfloat16().cuda().abs()
    if what == "scores of a piece":
        K[64 * ((n - 1) // 64):, :, 3] = float("-inf")
    else:
        V[-1, 0, 5] = float("inf")
    cache.append([(K, V)])
    got = cache.attend([q], 128 ** -0.5)[0].double()
    want = plain_attention(q, K, V, 128 ** -0.5, None) if what == "scores of a piece" else \
        plain_attention(q, K, V.nan_to_num(posinf=0.0), 128 ** -0.5, None)
    if what != "scores of a piece":
        want[0, 5] = float("inf")
    ok = torch.isclose(got, want, rtol=0, atol=1e-5 * V.double().nan_to_num(posinf=0.0).square().mean().sqrt().item())
    assert ok.all(), (got[~ok], want[~ok])


def test_attend_refuses_what_does_not_fit():
    from paper_2501_19392_amd import binding as B
    from paper_2501_19392_amd.cache import AquaKVCache
    lay = U.make_layers(1, "bf16", 16)[1]
    cache = AquaKVCache([lay], max_tokens=40, sink_tokens=4, buffer_tokens=8)
    kv = torch.randn(40, 1, 128).bfloat16().cuda()
    with pytest.raises(ValueError):
        cache.attend([kv[0].contiguous()], 1.0)                        # nothing cached
    cache.append([(kv, kv)])
    with pytest.raises(ValueError):
        cache.attend([kv[0].float()], 1.0)
    cache.attend([kv[0].contiguous()], 1.0)
    A = cache._attend
    for bad in (dict(n_sink=[5]), dict(n_compressed=[41]), dict(n_recent=[9]), dict(n_sink=[0], n_compressed=[0], n_recent=[0]),
                dict(workspace=A["ws"][:256])):
        args = dict(n_sink=[4], n_compressed=[32], n_recent=[4], workspace=A["ws"]) | bad
        with pytest.raises(B.AquaKVError):
            B.aquakv_attend_cache(A["layers"], A["shape"], score_scale=1.0, hat=A["hat"], **args)


@pytest.mark.parametrize("rht_group", [None, 1024])
@pytest.mark.parametrize("n", [1029, 1500, 1700, 2052, 2150, 3060, 3300])
def test_values_and_next_keys_recovered_together(n, rht_group):
    """Few compressed tokens: the values of a layer and the keys of the next one in one launch, on tiles of 64, 96, 128 and 192 rows (and
    not at all at the last length), layers of other quantizers and a 16-bit layer between them: the last two layers' recovered
    tensors have the bits of the sweep, and every layer the attention over the tensors of the sweep."""
    from paper_2501_19392_amd.cache import AquaKVCache
    print(f"case recovered together n={n} group={rht_group}", flush=True)
    H, QH, D = 8, 16, 1024
    gen = torch.Generator().manual_seed(n)
    kw = {"rht_group": rht_group} if rht_group else {}
    layers, kv, qs = [], [], []
    for l, points in enumerate((256, 16, 16, 64, None, 64, 64, 16)):
        w = [None, None] if l == 0 else [0.3 * torch.randn(D, d, generator=gen) / d ** 0.5 for d in (D, 2 * D)]
        layers.append(None if points is None else U.make_layers(H, "bf16", points, layer_idx=l, w_k=w[0], w_v=w[1], **kw)[1])
        kv.append(tuple(torch.randn(n, H, 128, generator=gen).bfloat16().cuda() for _ in range(2)))
        qs.append(torch.randn(QH, 128, generator=gen).bfloat16().cuda())
    for count in (len(layers), len(layers) - 1):             # the last layer behind a pair, and behind none
        cache = AquaKVCache(layers[:count], max_tokens=n, sink_tokens=4, buffer_tokens=64)
        cache.append(kv[:count])
        got = [o.clone() for o in cache.attend(qs[:count], 128 ** -0.5)]
        c = cache.n_compressed
        hat = [t[:c].clone() for t in cache._attend["hat"]]
        for l, K, V in cache.sweep():
            want = plain_attention(qs[l], K, V, 128 ** -0.5, None)
            assert float((got[l].double() - want).abs().max() / V.double().square().mean().sqrt()) < 1e-5, l
            if l >= count - 2:
                for a, b in zip(hat[2 * (l & 1):2 * (l & 1) + 2], (K[4:4 + c], V[4:4 + c])):
                    assert torch.equal(a.view(torch.int16), b.contiguous().view(torch.int16)), l


@pytest.mark.parametrize("H,QH,lengths,rht_group", [
    (8, 24, [69], None), (8, 8, [130, 700], 1024),              # two tensors on tiles of 32 and of 64 rows
    (8, 16, [1400], 1024), (8, 32, [2700], None),              # of 96 and of 192 rows
    (8, 24, [1800], 1024), (8, 32, [1100, 900], None),          # of 128 rows
    (3, 6, [8180], None),                                       # on 128 rows, more tiles than CUs
    (1, 3, [4229], None),                                       # 67 pieces, two to a workgroup: the last one has one
    (8, 64, [3300], 1024), (8, 32, [2600, 4, 2300], None)])     # one tensor on tiles of 128 and of 256 rows
def test_attention_beside_the_recovery_of_the_next_layer(H, QH, lengths, rht_group):
    """Two tensors: same bits as with attention in launches of its own, which a workspace without the third place for keys gives.  One
    tensor (the last two cases): the same call twice.  In every case attention over the tensors of the sweep."""
    from paper_2501_19392_amd import binding as B
    from paper_2501_19392_amd.cache import AquaKVCache
    print(f"case attention beside recovery H={H} QH={QH} lengths={lengths} group={rht_group}", flush=True)
    L, NB, n, D = 5, len(lengths), max(lengths), H * 128
    gen = torch.Generator().manual_seed(n)
    kw = {"rht_group": rht_group} if rht_group else {}
    layers, kv, qs = [], [], []
    for l in range(L):
        w = [None, None] if l == 0 else [0.3 * torch.randn(D, d, generator=gen) / d ** 0.5 for d in (D, 2 * D)]
        layers.append(U.make_layers(H, "bf16", 256 if l == 0 else 16, layer_idx=l, w_k=w[0], w_v=w[1], **kw)[1])
        kv.append(tuple(torch.randn(NB, n, H, 128, generator=gen).bfloat16().cuda() for _ in range(2)))
        qs.append(torch.randn(NB, QH, 128, generator=gen).bfloat16().cuda())
    cache = AquaKVCache(layers, max_tokens=n, sink_tokens=4, buffer_tokens=64, batch=NB)
    cache.append(kv, lengths=lengths)
    got = [o.clone() for o in cache.attend(qs, 128 ** -0.5)]
    compressed, row = sum(c for c in (cache.n_compressed if NB > 1 else [cache.n_compressed])), D * 2
    A = cache._attend
    third = -(-min(NB * cache._C, 192 // H * 128) * row // 256) * 256
    A["ws"] = A["ws"][:B.aquakv_attend_cache_workspace_bytes(A["layers"], A["shape"]) - third]
    one = (sum(-(-t // 64) for t in lengths) * QH * 130 * 4 + 255) // 256 * 256
    codec = max(lay.alloc_workspace(compressed).numel() for lay in layers)
    if compressed <= 192 // H * 128:                             # no room for the third place beside one layer's partial results
        A["ws"] = A["ws"][:(codec + 255) // 256 * 256 + one]
    again = [o.clone() for o in cache.attend(qs, 128 ** -0.5)]
    for l in range(L):
        assert torch.equal(got[l], again[l]), l
    for b in range(NB):
        for l, K, V in cache.sweep(b):
            want = plain_attention(qs[l][b], K, V, 128 ** -0.5, None)
            assert float((got[l][b].double() - want).abs().max() / V.double().square().mean().sqrt()) < 1e-5, (b, l)
