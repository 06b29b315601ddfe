"""aquakv_encode_layers: a stack of layers gives the bits of one aquakv_encode_layer call per layer (GPU), and faults in its arguments
are refused before the device is touched (CPU, made-up addresses)."""
import pytest
import torch

from paper_2501_19392_amd import binding as B
from tests import parity_utils as U
from tests.test_abi_cache_host import layer

MiB = 1 << 20
H, D = 8, 1024


class Stack:
    def __init__(self, layers, tokens=300):
        self.top, self.tokens = 1 << 40, tokens
        self.entries = [[lay, self.address(), self.address(), *(self.address() if lay is not None else 0 for _ in range(4))] for lay in layers]
        self.hat = [self.address() for _ in range(4)]
        self.workspace = self.address(64 * MiB)
        self.need = max([B.aquakv_workspace_bytes(lay, tokens) for lay in layers if lay is not None], default=0)

    def address(self, size=16 * MiB):
        self.top += size
        return self.top - size

    def status(self, workspace_bytes=None):
        with pytest.raises(B.AquaKVError) as e:
            B.aquakv_encode_layers(self.entries, self.tokens, self.hat, (self.workspace, self.need if workspace_bytes is None else workspace_bytes))
        return e.value.status


def test_faults_in_the_arguments_are_refused():
    stack = [layer(first=True), layer(), None, layer()]
    assert Stack([layer()]).status() == B.AQUAKV_ENULL                       # predictors, but no layer before
    assert Stack([layer(first=True), layer(d_in_k=128)]).status() == B.AQUAKV_EINVAL
    assert Stack([layer(first=True), layer(d_in_v=D + 128)]).status() == B.AQUAKV_EINVAL
    assert Stack([layer(first=True), layer(dtype=B.AQUAKV_FP32)]).status() == B.AQUAKV_EINVAL
    assert Stack(stack, tokens=-1).status(0) == B.AQUAKV_EINVAL
    s = Stack(stack)
    assert s.status(s.need - 1) == B.AQUAKV_EWORKSPACE
    for field in (1, 3, 6):                                                  # K, k_codes, v_scales
        s = Stack(stack)
        s.entries[1][field] = 0
        assert s.status() == B.AQUAKV_ENULL
        s.entries[1][field] = (1 << 50) + (1 if field == 6 else 2)
        assert s.status() == B.AQUAKV_EALIGN
    s = Stack(stack)
    s.hat[2] = 0
    assert s.status() == B.AQUAKV_ENULL
    for a, b in (((0, 3), (1, 5)), ((1, 3), (2, 1)), ((3, 4), (3, 2))):      # codes over another layer's codes, its input, their own
        s = Stack(stack)
        s.entries[a[0]][a[1]] = s.entries[b[0]][b[1]]
        assert s.status() == B.AQUAKV_EINVAL
    for other in (1, 3):                                                     # hat over a layer's values, over itself
        s = Stack(stack)
        s.hat[0] = s.entries[3][2] if other == 1 else s.hat[3]
        assert s.status() == B.AQUAKV_EINVAL
    s = Stack(stack)
    s.workspace = s.entries[1][1]
    assert s.status() == B.AQUAKV_EINVAL
    s = Stack(stack, tokens=0)                                               # nothing to do
    B.aquakv_encode_layers(s.entries, 0, s.hat, (s.workspace, s.need))


PARAMETERS = dict(w_k=D * D * 2, w_v=2 * D * D * 2, b_k=4 * D, b_v=4 * D, signs_k=D, signs_v=D, codebook=16 * 8,
                  search_table=B.aquakv_search_table_bytes(16))


@pytest.mark.parametrize("written", ["hat", "workspace", "k_codes", "v_scales"])
@pytest.mark.parametrize("name", PARAMETERS)
def test_nothing_is_written_over_the_parameters(name, written):
    """The last bytes of a layer's parameter at the first byte of a buffer that the call writes, in the next layer and in one further on."""
    for owner in (2, 4):
        s = Stack([layer(first=True), *(layer() for _ in range(4))])
        at = {"hat": s.hat[1], "workspace": s.workspace, "k_codes": s.entries[1][3], "v_scales": s.entries[1][6]}[written]
        s.entries[owner][0] = layer(**{name: at - PARAMETERS[name] // 16 * 16 + 16})
        assert s.status() == B.AQUAKV_EINVAL, owner
        assert f"{name} of layer {owner}" in B.aquakv_last_error() and "overlaps" in B.aquakv_last_error()


@pytest.mark.gpu
@pytest.mark.parametrize("rht_group", [None, 1024])
@pytest.mark.parametrize("tokens", [1, 31, 512, 513, 1025, 1536, 1537, 2049, 3072, 3073, 4096, 4097])
def test_a_stack_has_the_bits_of_its_layers(tokens, rht_group):
    """Both sides of the lines between tiles of 32 to 192 rows and launches of one tensor; layers of other quantizers, a 16-bit
    layer and one without predictors in between; grids of their own and a common one; with the least workspace and with room for more."""
    print(f"case encode stack tokens={tokens} group={rht_group}", flush=True)
    gen = torch.Generator().manual_seed(tokens)
    kw = {"rht_group": rht_group} if rht_group else {}
    layers, kv = [], []
    for l, (points, predictor) in enumerate([(256, False), (16, True), (16, True), (16, True), (64, True), (None, False), (64, True),
                                             (2, True), (2, True), (16, False)]):
        w = [0.3 * torch.randn(D, d, generator=gen) / d ** 0.5 for d in (D, 2 * D)] if predictor else [None, None]
        b = torch.randn(D, generator=gen) if l == 2 else None
        q = dict(rtn_bits=2) if points == 2 else {}
        lay = None if points is None else U.make_layers(H, "bf16", 16 if points == 2 else points, layer_idx=l, w_k=w[0], w_v=w[1],
                                                         b_v=b, **kw, **q)[1]
        if l == 3:                                               # the grid of the layer before
            lay.codebook, lay.search_table = layers[2].codebook, layers[2].search_table
            lay.c.codebook, lay.c.search_table = layers[2].c.codebook, layers[2].c.search_table
        layers.append(lay)
        kv.append(tuple(torch.randn(tokens, H, 128, generator=gen).bfloat16().cuda() for _ in range(2)))
    new = lambda: [None if lay is None else [t.zero_() for p in (lay.alloc_codes(tokens), lay.alloc_codes(tokens)) for t in p] for lay in layers]
    least = max(B.aquakv_workspace_bytes(lay, tokens) for lay in layers if lay is not None)
    want, Kp, Vp, hats = new(), None, None, []
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    for lay, (K, V), out in zip(layers, kv, want):
        if lay is None:
            Kp, Vp = K, V
            hats.append(None)
            continue
        Kh, Vh = lay.alloc_kv(tokens), lay.alloc_kv(tokens)
        B.aquakv_encode_layer(lay, tokens, K, V, Kp if lay.c.d_in_k else None, Vp if lay.c.d_in_v else None, *out, Kh, Vh, ws)
        Kp, Vp = Kh, Vh
        hats.append((Kh, Vh))
    some = next(lay for lay in layers if lay is not None)
    for room in (least, least + 2 * tokens * D * 2):
        got, hat = new(), [some.alloc_kv(tokens) for _ in range(4)]
        B.aquakv_encode_layers([(lay, K, V, *(out or (None,) * 4)) for lay, (K, V), out in zip(layers, kv, got)], tokens, hat,
                               torch.empty(room, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        for l, (a, b) in enumerate(zip(got, want)):
            assert a is None or all(torch.equal(x, y) for x, y in zip(a, b)), (l, room)
        for l in (len(layers) - 2, len(layers) - 1):
            for x, y in zip(hat[2 * (l & 1):2 * (l & 1) + 2], hats[l]):
                assert torch.equal(x.view(torch.int16), y.view(torch.int16)), (l, room)


@pytest.mark.gpu
@pytest.mark.parametrize("tokens", [768, 769, 1344, 1345, 1536, 2016, 2017, 2432, 2433])
def test_predictions_of_two_tensors_on_tiles_of_two_sizes(tokens):
    """Both sides of the lines between the pairs of sizes (groups across the heads)."""
    test_a_stack_has_the_bits_of_its_layers(tokens, 1024)
