"""Tiles of 32, 64, 96, 128, 192 and 320 token rows (short ranges, and ranges that leave a round of the large tiles nearly empty):
encode, decode and the scoring call against the stage calls (aquakv_predict, aquakv_quantize, aquakv_dequantize), bit for
bit, at the edges of every tile, with and without bias, for predictors as narrow as two k-tiles, all quantizers and both groupings."""
import pytest
import torch

from tests import parity_utils as U

pytestmark = pytest.mark.gpu
bits = lambda t: t.contiguous().view(torch.uint8)


def layer(H, dk, quantizer, rht_group=None, bias=True):
    D = H * 128
    kw = dict(rtn_bits=int(quantizer[3:])) if quantizer.startswith("rtn") else {}
    if rht_group:
        kw["rht_group"] = rht_group
    n = 16 if quantizer.startswith("rtn") else int(quantizer[1:])
    g = torch.Generator().manual_seed(6)
    bk, bv = (torch.randn(D, generator=g) * 0.3 if bias else None for _ in range(2))
    return U.make_layers(H, "bf16", n, layer_idx=1, w_k=U.random_weights(D, dk, 21, 0.7),
                         w_v=U.random_weights(D, dk + D, 22, 0.7), b_k=bk, b_v=bv, **kw)[1]


CASES = [(8, 1024, T) for T in (1, 31, 33, 1024, 1025, 1089, 2048, 2049, 2177, 2976, 3071, 3072, 3073, 4096, 4097, 4289, 6144, 6145, 8449)] + [
    (3, 128, 2700), (3, 128, 33), (16, 256, 700), (1, 384, 8200), (8, 192 * 2, 129)]


@pytest.mark.parametrize("H,dk,T", CASES)
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("n64", None), ("n256", None), ("rtn2", None), ("rtn4", None),
                                                 ("n16", 1024), ("n64", 1024), ("rtn4", 1024)])
def test_tiles_give_the_bits_of_the_stage_calls(H, dk, T, quantizer, rht_group):
    from paper_2501_19392_amd import binding as B
    if rht_group and H != 8:
        pytest.skip("groups across heads are built for 8 heads")
    print(f"case tiles H={H} dk={dk} T={T} {quantizer} group={rht_group}", flush=True)
    lg, D = layer(H, dk, quantizer, rht_group, bias=T % 2 == 1), H * 128
    g = torch.Generator(device="cuda").manual_seed(300 + T)
    mk = lambda w: torch.randn(T, w, generator=g, device="cuda").bfloat16()
    K, V = mk(D).view(T, H, 128), mk(D).view(T, H, 128)
    Kp, Vp = mk(dk), mk(dk)
    poison = lambda *ts: [t.view(torch.uint8).fill_(0xAB) for t in ts]
    (kc, ks), (vc, vs) = lg.alloc_codes(T), lg.alloc_codes(T)
    Kh, Vh, Kd, Vd = (lg.alloc_kv(T) for _ in range(4))
    poison(kc, ks, vc, vs, Kh, Vh, Kd, Vd)
    ws = lg.alloc_workspace(T)
    B.aquakv_encode_layer(lg, T, K, V, Kp, Vp, kc, ks, vc, vs, Kh, Vh, ws)
    B.aquakv_decode_layer(lg, T, kc, ks, vc, vs, Kp, Vp, Kd, Vd, ws)
    P = torch.empty(T, D, dtype=torch.float32, device="cuda")
    for which, x0, x1, X, codes, scales, hat, dec in ((B.AQUAKV_KEY, Kp, None, K, kc, ks, Kh, Kd),
                                                      (B.AQUAKV_VALUE, Vp, Kh, V, vc, vs, Vh, Vd)):
        c2, s2 = lg.alloc_codes(T)
        h2, d2 = lg.alloc_kv(T), lg.alloc_kv(T)
        B.aquakv_predict(lg, which, T, x0, x1, P)
        B.aquakv_quantize(lg, which, T, X, P, c2, s2, h2)
        B.aquakv_dequantize(lg, which, T, c2, s2, P, d2)
        torch.cuda.synchronize()
        for name, a, b in (("codes", codes, c2), ("scales", scales, s2), ("encode", hat, h2), ("decode", dec, d2)):
            assert torch.equal(bits(a), bits(b)), (which, name)


@pytest.mark.parametrize("T", [1, 1024, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("quantizer", ["n16", "n256", "rtn2"])
def test_groups_across_heads_whatever_the_workspace_holds(T, quantizer):
    """Encode with the predictions in pieces (the required workspace), in one piece (a larger one), and with the temporary keys in
    the workspace too: the same codes, equal to those of the stage calls; nothing behind the workspace is touched."""
    from paper_2501_19392_amd import binding as B
    print(f"case wide workspace T={T} {quantizer}", flush=True)
    lg, D = layer(8, 1024, quantizer, 1024, bias=T % 2 == 1), 1024
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V, Kp, Vp = (torch.randn(T, D, generator=g, device="cuda").bfloat16() for _ in range(4))
    P = torch.empty(T, D, dtype=torch.float32, device="cuda")
    (kc, ks), (vc, vs) = lg.alloc_codes(T), lg.alloc_codes(T)
    Kh, Vh = lg.alloc_kv(T), lg.alloc_kv(T)
    for which, x0, x1, X, c, s, hat in ((B.AQUAKV_KEY, Kp, None, K, kc, ks, Kh), (B.AQUAKV_VALUE, Vp, Kh, V, vc, vs, Vh)):
        B.aquakv_predict(lg, which, T, x0, x1, P)
        B.aquakv_quantize(lg, which, T, X, P, c, s, hat)
    want = [bits(t) for t in (kc, ks, vc, vs, Vh, Kh)]
    need = lg.alloc_workspace(T).numel()
    for extra in (0, 1040, 3 * T * D, 5 * T * D + (8 << 20)):
        for with_keys in (True, False):
            arena = torch.full((need + extra + 4096,), 0xCD, dtype=torch.uint8, device="cuda")
            (kc, ks), (vc, vs) = lg.alloc_codes(T), lg.alloc_codes(T)
            Kh, Vh = lg.alloc_kv(T), lg.alloc_kv(T)
            B.aquakv_encode_layer(lg, T, K, V, Kp, Vp, kc, ks, vc, vs, Kh if with_keys else None, Vh, arena[:need + extra])
            torch.cuda.synchronize()
            for name, a, b in zip(("k_codes", "k_scales", "v_codes", "v_scales", "Vhat", "Khat"), (kc, ks, vc, vs, Vh, Kh), want):
                assert (name == "Khat" and not with_keys) or torch.equal(bits(a), b), (extra, with_keys, name)
            assert bool((arena[need + extra:] == 0xCD).all())


@pytest.mark.parametrize("H,dk,batch,S", [(8, 1024, 1, 1), (8, 1024, 3, 33), (8, 1024, 5, 100), (8, 1024, 2, 1000),
                                          (8, 1024, 2, 1100), (8, 1024, 3, 1100), (8, 1024, 5, 1100), (8, 1024, 1, 8449), (3, 128, 2, 65)])
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("rtn2", None), ("n256", 1024)])
def test_scores_of_a_batch_are_those_of_its_sequences(H, dk, batch, S, quantizer, rht_group):
    from paper_2501_19392_amd import binding as B
    if rht_group and H != 8:
        pytest.skip("groups across heads are built for 8 heads")
    print(f"case tile scores H={H} batch={batch} S={S} {quantizer} group={rht_group}", flush=True)
    lg, D, T, QH = layer(H, dk, quantizer, rht_group, bias=S % 2 == 1), H * 128, batch * S, 4 * H
    g = torch.Generator(device="cuda").manual_seed(70 + T)
    K = torch.randn(T, H, 128, generator=g, device="cuda").bfloat16()
    Kp = torch.randn(T, dk, generator=g, device="cuda").bfloat16()
    q = torch.randn(batch, QH, 128, generator=g, device="cuda").bfloat16()
    ang = torch.arange(S, device="cuda")[:, None] * 0.3 ** torch.arange(64, device="cuda")[None]
    cos, sin = ang.cos().float().contiguous(), ang.sin().float().contiguous()
    kc, ks = lg.alloc_codes(T)
    Kh, Ko, ws = lg.alloc_kv(T), lg.alloc_kv(T), lg.alloc_workspace(T)
    B.aquakv_encode_keys(lg, T, K, Kp, kc, ks, Kh, ws)
    for rope in (None, (cos, sin)):
        got = torch.full((batch, QH, S), float("nan"), device="cuda")
        call = (lambda n, c, s, p, qq, out, ko: B.aquakv_decode_attn_scores(lg, n, S, QH, c, s, p, qq, 0.125, out, ko, ws)) if rope is None \
            else (lambda n, c, s, p, qq, out, ko: B.aquakv_decode_attn_scores_rope(lg, n, S, QH, c, s, p, qq, cos, sin, 0.125, out, ko, ws))
        call(batch, kc, ks, Kp, q, got, Ko)
        torch.cuda.synchronize()
        assert torch.equal(bits(Ko), bits(Kh))
        keys = Kh.float().view(batch, S, H, 128)
        if rope is not None:
            a, b = keys[..., :64], keys[..., 64:]
            c, s = cos[None, :, None], sin[None, :, None]
            keys = torch.cat([a * c - b * s, b * c + a * s], -1)
        want = (q.float().view(batch, H, 4, 1, 128) * keys.permute(0, 2, 1, 3)[:, :, None]).sum(-1).view(batch, QH, S) * 0.125
        assert torch.allclose(got, want, rtol=1e-4, atol=1e-4 * want.abs().max().item())
        for i in range(batch):
            one = torch.empty(1, QH, S, device="cuda")
            rows = slice(i * S, (i + 1) * S)
            call(1, kc[rows].clone(), ks[rows].clone(), Kp[rows].clone(), q[i:i + 1].clone(), one, None)
            torch.cuda.synchronize()
            assert torch.equal(one[0], got[i]), i


@pytest.mark.parametrize("name", ["w_k", "w_v", "b_k", "b_v", "codebook", "signs_k", "signs_v", "search_table"])
def test_parameters_behind_the_needed_workspace_are_left_alone(name):
    """One arena: the workspace is stated as all that is left of it, and a parameter of the layer lies in that rest."""
    from paper_2501_19392_amd import binding as B
    T, D = 2100, 1024                                  # does not fit the needed workspace in one piece
    print(f"case arena with {name}", flush=True)
    lg = layer(8, 1024, "n16", 1024)
    if lg.search_table is None:
        lg.search_table = B.build_search_table(lg.codebook)
        lg.c.search_table = lg.search_table.data_ptr()
    g = torch.Generator(device="cuda").manual_seed(5)
    K, V, Kp, Vp = (torch.randn(T, D, generator=g, device="cuda").bfloat16() for _ in range(4))

    def encode(workspace, khat):
        codes = [t for _ in range(2) for t in lg.alloc_codes(T)]
        Kh, Vh = lg.alloc_kv(T), lg.alloc_kv(T)
        B.aquakv_encode_layer(lg, T, K, V, Kp, Vp, *codes, Kh if khat else None, Vh, workspace)
        torch.cuda.synchronize()
        return codes + [Vh]

    want = encode(lg.alloc_workspace(T), True)
    x = bits(getattr(lg, name)).flatten()
    need = lg.alloc_workspace(T).numel()
    for khat, at in ((True, need), (False, need), (False, need + (4 << 20))):
        arena = torch.zeros(need + (12 << 20), dtype=torch.uint8, device="cuda")
        arena[at:at + x.numel()] = x
        setattr(lg.c, name, arena.data_ptr() + at)
        got = encode(arena, khat)
        assert torch.equal(arena[at:at + x.numel()], x)
        for a, b in zip(got, want, strict=True):
            assert torch.equal(bits(a), bits(b))
        setattr(lg.c, name, getattr(lg, name).data_ptr())


@pytest.mark.parametrize("name,T,rht_group", [("b_v", 2100, 1024), ("w_v", 2100, 1024), ("w_k", 19000, 1024), ("search_table", 5000, 1024),
                                              ("b_v", 300, None), ("codebook", 300, 1024)])
def test_parameters_in_the_room_of_a_temporary_khat_are_left_alone(name, T, rht_group):
    """With a Khat to write to, the workspace's room for a temporary one is not needed: a parameter of the layer may lie there, and
    neither predictions nor sums of the call are put over it."""
    from paper_2501_19392_amd import binding as B
    D = 1024
    print(f"case {name} in the room of Khat, T={T} group={rht_group}", flush=True)
    lg = layer(8, 1024, "n16", rht_group)
    if lg.search_table is None:
        lg.search_table = B.build_search_table(lg.codebook)
        lg.c.search_table = lg.search_table.data_ptr()
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V, Kp, Vp = (torch.randn(T, D, generator=g, device="cuda").bfloat16() for _ in range(4))

    def encode_decode(workspace):
        codes = [t for _ in range(2) for t in lg.alloc_codes(T)]
        hats = [lg.alloc_kv(T) for _ in range(4)]
        B.aquakv_encode_layer(lg, T, K, V, Kp, Vp, *codes, *hats[:2], workspace)
        B.aquakv_decode_layer(lg, T, *codes, Kp, Vp, *hats[2:], workspace)
        torch.cuda.synchronize()
        return codes + hats

    want = encode_decode(lg.alloc_workspace(T))
    x = bits(getattr(lg, name)).flatten()
    arena = torch.zeros(B.aquakv_workspace_bytes(lg, T), dtype=torch.uint8, device="cuda")
    at = arena.numel() - T * D * 2                     # behind the weights in another order, where there are such
    arena[at:at + x.numel()] = x
    setattr(lg.c, name, arena.data_ptr() + at)
    got = encode_decode(arena)
    assert torch.equal(arena[at:at + x.numel()], x)
    for a, b in zip(got, want, strict=True):
        assert torch.equal(bits(a), bits(b))


@pytest.mark.parametrize("T", [1, 130, 511, 512, 513])
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("n64", None), ("rtn4", None), ("n256", 1024)])
def test_keys_and_values_of_few_rows_at_once(T, quantizer, rht_group):
    """Up to 512 rows of 8 heads the keys' launch takes half of the values' product along, whose sums wait in the workspace and in
    Vhat: the bits of the halves called one after the other, which do not run that way, for every choice of outputs (without Khat,
    or with Vhat over V, the layer call does not either), and the least workspace there may be, with parameters behind it."""
    from paper_2501_19392_amd import binding as B
    print(f"case at once T={T} {quantizer} group={rht_group}", flush=True)
    lg, D = layer(8, 1024, quantizer, rht_group, bias=T % 2 == 1), 1024
    g = torch.Generator(device="cuda").manual_seed(900 + T)
    K, V, Kp, Vp = (torch.randn(T, 8, 128, generator=g, device="cuda").bfloat16() for _ in range(4))
    need = B.aquakv_workspace_bytes(lg, T)
    new = lambda: [*lg.alloc_codes(T), *lg.alloc_codes(T)]
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    want, Kh, Vh = new(), lg.alloc_kv(T), lg.alloc_kv(T)
    B.aquakv_encode_keys(lg, T, K, Kp, want[0], want[1], Kh, ws)
    B.aquakv_encode_values(lg, T, V, Vp, Kh, want[2], want[3], Vh, ws)
    arena = torch.full((need + lg.w_v.numel() * 2,), 0xCD, dtype=torch.uint8, device="cuda")
    arena[need:] = bits(lg.w_v).flatten()
    lg.c.w_v = arena.data_ptr() + need
    for keys, values in (("own", "own"), ("own", "in place"), ("in place", "own"), (None, "own"), ("own", None)):
        got, k, v = new(), K.clone(), V.clone()
        kh = {"own": lg.alloc_kv(T), "in place": k, None: None}[keys]
        vh = {"own": lg.alloc_kv(T), "in place": v, None: None}[values]
        B.aquakv_encode_layer(lg, T, k, v, Kp, Vp, *got, kh, vh, arena[:need])
        torch.cuda.synchronize()
        for a, b in list(zip(got, want)) + [(kh, Kh), (vh, Vh)]:
            assert a is None or torch.equal(bits(a), bits(b)), (keys, values)
    for size in (need, arena.numel()):                # (the rest of the arena stated too: the parameter in it stays)
        kd, vd = lg.alloc_kv(T), lg.alloc_kv(T)
        B.aquakv_decode_layer(lg, T, *want, Kp, Vp, kd, vd, arena[:size])
        torch.cuda.synchronize()
        assert torch.equal(bits(kd), bits(Kh)) and torch.equal(bits(vd), bits(Vh))
    assert torch.equal(arena[need:], bits(lg.w_v).flatten())


@pytest.mark.parametrize("T", [2049, 12288, 12289, 16384, 16417])
@pytest.mark.parametrize("quantizer", ["n16", "n64", "rtn2"])
def test_groups_across_heads_over_the_rounds_of_whole_tokens(T, quantizer):
    """Long ranges: rounds of the kernel that owns whole tokens, and the rows left over from predictions whose halves lie in the
    workspace and in the rows of the reconstruction (its own, over the input, or none): the bits of the stage calls."""
    from paper_2501_19392_amd import binding as B
    print(f"case wide rounds T={T} {quantizer}", flush=True)
    lg, D = layer(8, 1024, quantizer, 1024, bias=T % 2 == 1), 1024
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V, Kp, Vp = (torch.randn(T, 8, 128, generator=g, device="cuda").bfloat16() for _ in range(4))
    P = torch.empty(T, D, dtype=torch.float32, device="cuda")
    new = lambda: [*lg.alloc_codes(T), *lg.alloc_codes(T)]
    want, Kh, Vh = new(), lg.alloc_kv(T), lg.alloc_kv(T)
    for which, x0, x1, X, c, s, hat in ((B.AQUAKV_KEY, Kp, None, K, *want[:2], Kh), (B.AQUAKV_VALUE, Vp, Kh, V, *want[2:], Vh)):
        B.aquakv_predict(lg, which, T, x0, x1, P)
        B.aquakv_quantize(lg, which, T, X, P, c, s, hat)
    need = B.aquakv_workspace_bytes(lg, T)
    for keys, values in (("own", "own"), ("in place", "own"), ("own", "in place"), (None, None)):
        arena = torch.full((need + 4096,), 0xCD, dtype=torch.uint8, device="cuda")
        got, k, v = new(), K.clone(), V.clone()
        kh = {"own": lg.alloc_kv(T), "in place": k, None: None}[keys]
        vh = {"own": lg.alloc_kv(T), "in place": v, None: None}[values]
        B.aquakv_encode_layer(lg, T, k, v, Kp, Vp, *got, kh, vh, arena[:need])
        torch.cuda.synchronize()
        for a, b in list(zip(got, want)) + [(kh, Kh), (vh, Vh)]:
            assert a is None or torch.equal(bits(a), bits(b)), (keys, values)
        assert bool((arena[need:] == 0xCD).all())
    kh = lg.alloc_kv(T)                               # the halves, with the least workspace they need
    got, ws = new(), torch.empty(D * 2 * D * 2, dtype=torch.uint8, device="cuda")
    B.aquakv_encode_keys(lg, T, K, Kp, got[0], got[1], kh, ws)
    B.aquakv_encode_values(lg, T, V, Vp, kh, got[2], got[3], None, ws)
    torch.cuda.synchronize()
    assert all(torch.equal(bits(a), bits(b)) for a, b in zip(got, want)) and torch.equal(bits(kh), bits(Kh))


@pytest.mark.parametrize("T,quantizer,keys,values,split", [
    (8192, "n16", "in place", "in place", True), (8193, "n16", "in place", "in place", False),        # two pieces
    (7168, "rtn2", "in place", "in place", True), (7169, "rtn2", "in place", "in place", False),
    (11000, "n256", "in place", None, False), (16384 + 4097, "rtn4", "own", "own", False), (16384 + 4096, "rtn4", "own", "own", True),
    (6144, "n64", None, "own", True), (6145, "n64", None, "own", False)])                             # three pieces, four
def test_groups_across_heads_in_several_pieces(T, quantizer, keys, values, split):
    """Where the workspace holds the predictions of few rows only, pieces of them are taken up to the range where a round of whole
    tokens costs less: beyond it nothing is written behind the weights and the temporary Khat.  The bits of the stage calls either way."""
    from paper_2501_19392_amd import binding as B
    print(f"case pieces T={T} {quantizer} keys={keys} values={values}", flush=True)
    lg, D = layer(8, 1024, quantizer, 1024, bias=T % 2 == 1), 1024
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V, Kp, Vp = (torch.randn(T, 8, 128, generator=g, device="cuda").bfloat16() for _ in range(4))
    P = torch.empty(T, D, dtype=torch.float32, device="cuda")
    new = lambda: [*lg.alloc_codes(T), *lg.alloc_codes(T)]
    want, Kh, Vh = new(), lg.alloc_kv(T), lg.alloc_kv(T)
    for which, x0, x1, X, c, s, hat in ((B.AQUAKV_KEY, Kp, None, K, *want[:2], Kh), (B.AQUAKV_VALUE, Vp, Kh, V, *want[2:], Vh)):
        B.aquakv_predict(lg, which, T, x0, x1, P)
        B.aquakv_quantize(lg, which, T, X, P, c, s, hat)
    arena = torch.full((B.aquakv_workspace_bytes(lg, T),), 0xCD, dtype=torch.uint8, device="cuda")
    got, kh, vh = new(), {"own": Kh.clone(), "in place": K.clone(), None: None}[keys], {"own": Vh.clone(), "in place": V.clone(), None: None}[values]
    k, v = (kh if keys == "in place" else K), (vh if values == "in place" else V)
    B.aquakv_encode_layer(lg, T, k, v, Kp, Vp, *got, kh, vh, arena)
    torch.cuda.synchronize()
    for a, b in list(zip(got, want)) + [(kh, Kh), (vh, Vh)]:
        assert a is None or torch.equal(bits(a), bits(b))
    weights = D * 2 * D * 2                                # the predictors' in the order of the encoder's main loop
    if keys is None:                                       # behind them the temporary Khat: the predictions lie among the weights'
        hat = arena[weights:weights + T * D * 2].view(torch.int16).view(T, 8, 128)
        assert torch.equal(hat, Kh.view(torch.int16))
        lay = lg.w_v.flatten().view(torch.int16)
        sorted_front = arena[:weights].view(torch.int16).sort().values
        assert torch.equal(sorted_front, lay.sort().values) != split
    else:
        assert bool((arena[weights:] != 0xCD).any()) == split


@pytest.mark.parametrize("H,T", [(8, 4097), (8, 6500), (8, 9000), (3, 14000), (16, 3300), (6, 9001)])
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("n256", 1024), ("rtn4", None)])
def test_stand_alone_quantizer_in_more_workgroups_than_are_resident(H, T, quantizer, rht_group):
    """Head counts that a workgroup's 32 groups are and are not a multiple of, token counts that deal rounds out unevenly: the bits of calls
    of 512 tokens, whose workgroups have one round each."""
    from paper_2501_19392_amd import binding as B
    if rht_group and H != 8:
        pytest.skip("groups across heads are built for 8 heads")
    print(f"case quantizer rounds H={H} T={T} {quantizer} group={rht_group}", flush=True)
    kw = dict(rtn_bits=4) if quantizer == "rtn4" else {}
    if rht_group:
        kw["rht_group"] = rht_group
    lg = U.make_layers(H, "bf16", 16 if kw.get("rtn_bits") else int(quantizer[1:]), **kw)[1]
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = (torch.randn(T, H, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    got, want = ([*lg.alloc_codes(T), *lg.alloc_codes(T), lg.alloc_kv(T), lg.alloc_kv(T)] for _ in range(2))
    for t in got + want:
        t.view(torch.uint8).fill_(0xAB)
    ws = lg.alloc_workspace(T)
    B.aquakv_encode_layer(lg, T, K, V, None, None, *got, ws)
    for a in range(0, T, 512):
        n = min(512, T - a)
        B.aquakv_encode_layer(lg, n, K[a:a + n], V[a:a + n], None, None, *(t[a:a + n] for t in want), ws)
    torch.cuda.synchronize()
    for name, a, b in zip(("k codes", "k scales", "v codes", "v scales", "K", "V"), got, want):
        assert torch.equal(bits(a), bits(b)), name


@pytest.mark.parametrize("H,dk,T", [(8, 256, 10241), (8, 128, 12288), (8, 128, 12289), (8, 128, 16385), (8, 128, 18432), (8, 128, 18433), (4, 256, 33000),
                                    (3, 128, 29000)])
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("rtn2", None), ("n16", 1024), ("n64", 1024)])
def test_tiles_of_192_rows_in_several_rounds(H, dk, T, quantizer, rht_group):
    test_tiles_give_the_bits_of_the_stage_calls(H, dk, T, quantizer, rht_group)


@pytest.mark.parametrize("batch,S", [(16, 1100), (3, 3500)])
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("n256", 1024)])
def test_scores_on_tiles_of_192_rows_in_several_rounds(batch, S, quantizer, rht_group):
    test_scores_of_a_batch_are_those_of_its_sequences(8, 128, batch, S, quantizer, rht_group)


@pytest.mark.parametrize("H,dk,T", [(8, 128, 1500), (8, 128, 2500), (8, 128, 3500), (8, 128, 5000), (8, 128, 9000),      # two k-tiles, fewer than LDS holds
                                    (8, 128, 8191), (8, 128, 8192),                # from 16 MiB on rows are written past the L2s
                                    (5, 128, 1500), (12, 256, 900), (8, 256, 3600), (2, 128, 20000)])      # row blocks and heads that the XCDs share unevenly
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("n256", 1024)])
def test_tiles_of_short_products_and_uneven_shares(H, dk, T, quantizer, rht_group):
    test_tiles_give_the_bits_of_the_stage_calls(H, dk, T, quantizer, rht_group)


@pytest.mark.parametrize("H,dk,T", [(8, 128, 10241), (8, 256, 12288), (8, 128, 16385), (8, 128, 32769), (8, 128, 36864), (24, 128, 3201)])
@pytest.mark.parametrize("quantizer,rht_group", [("n16", None), ("n64", 1024), ("n256", 1024), ("rtn2", None), ("rtn4", 1024)])
def test_ranges_that_rounds_of_192_rows_cost_least_for(H, dk, T, quantizer, rht_group):
    test_tiles_give_the_bits_of_the_stage_calls(H, dk, T, quantizer, rht_group)


@pytest.mark.parametrize("batch,S,quantizer,rht_group", [(16, 1100, "n16", 1024), (3, 3500, "n16", 1024), (16, 1100, "rtn2", 1024), (5, 3300, "n256", 1024),
                                                         (3, 3500, "n64", 1024), (5, 3300, "n64", None), (5, 3300, "rtn2", None)])
def test_scores_on_192_rows_in_several_rounds(batch, S, quantizer, rht_group):
    test_scores_of_a_batch_are_those_of_its_sequences(8, 128, batch, S, quantizer, rht_group)
