"""Host-side checks of the calls of the cache manager (aquakv_attend_cache, aquakv_copy_ranges): bad arguments are refused before the
device is touched.  No GPU needed: the addresses are made up and never dereferenced."""
import pytest

from paper_2501_19392_amd import binding as B

MiB = 1 << 20
H, QH, D = 8, 32, 1024
CAP, SINKS, RECENT = 256, 4, 128
FIELDS = ("k_codes", "k_scales", "v_codes", "v_scales")


def layer(first=False, **kw):
    base = 0x10000                                        # parameters: apart from all other addresses, never read here
    d = dict(kv_heads=H, head_dim=128, vq_dim=2, n_codewords=16, dtype=B.AQUAKV_BF16, d_in_k=0 if first else D,
             d_in_v=0 if first else 2 * D, rht_group=0, codebook=base, signs_k=base, signs_v=base, w_k=base, b_k=None, w_v=base,
             b_v=None, search_table=None)
    d.update(kw)
    return B.aquakv_layer(**d)


class Call:
    """The arguments of an aquakv_attend_cache call over `layers`, every buffer 16 MiB of addresses of its own."""
    def __init__(self, layers, batch=2):
        self.top = 1 << 40
        self.batch = batch
        self.shape = B.aquakv_cache_shape(B.AQUAKV_BF16, H, QH, batch, SINKS, RECENT, CAP)
        entries = []
        for lay in layers:
            names = [*FIELDS, *("staged_" + n for n in FIELDS)] if lay is not None else ["raw_k", "raw_v"]
            names += ["sink_k", "sink_v", "recent_k", "recent_v", "q", "out"]
            entries.append((lay, {n: self.address() for n in names}))
        self.layers = B.cache_layers(entries)
        self.hat = [self.address() for _ in range(4)]
        self.need = B.aquakv_attend_cache_workspace_bytes(self.layers, self.shape)
        self.workspace = self.address(64 * MiB)
        self.counts = dict(n_sink=[SINKS] * batch, n_compressed=[128] * batch, n_recent=[7] * batch)
        self.rope = (self.address(), self.address())

    def address(self, size=16 * MiB):
        self.top += size
        return self.top - size

    def status(self, workspace_bytes=None, **counts):
        with pytest.raises(B.AquaKVError) as e:
            B.aquakv_attend_cache(self.layers, self.shape, **(self.counts | counts), score_scale=1.0, hat=self.hat,
                                  workspace=(self.workspace, self.need if workspace_bytes is None else workspace_bytes),
                                  rope_cos=self.rope[0], rope_sin=self.rope[1])
        return e.value.status


@pytest.mark.parametrize("kw", [dict(d_in_k=2 * D), dict(d_in_k=128), dict(d_in_v=3 * D), dict(d_in_v=D + 128), dict(d_in_k=0, d_in_v=3 * D)])
def test_predictors_of_another_width_than_the_cache_are_refused(kw):
    """They would read beyond the rows that the call itself lays out."""
    c = Call([layer(first=True), layer(**kw)])
    assert c.need == 0
    assert c.status(workspace_bytes=64 * MiB) == B.AQUAKV_EINVAL
    assert Call([layer(first=True), layer()]).need > 0 and Call([layer(first=True), layer(d_in_k=0)]).need > 0


def test_a_first_layer_with_predictors_is_refused_before_any_launch():
    c = Call([layer(), layer()])
    assert c.status() == B.AQUAKV_ENULL and "layer 0" in B.aquakv_last_error()


WRITTEN = ["out", "staged_k_codes", "staged_k_scales", "staged_v_codes", "staged_v_scales"]
READ = ["q", "sink_k", "sink_v", "recent_k", "recent_v", "k_codes", "k_scales", "v_codes", "v_scales", "raw_k", "raw_v"]


def stack():
    return Call([layer(first=True), None, layer()])


@pytest.mark.parametrize("written", WRITTEN + ["hat0", "hat1", "hat2", "hat3", "workspace"])
@pytest.mark.parametrize("other", WRITTEN + READ + ["hat0", "hat3", "workspace", "rope0", "rope1"])
def test_what_is_written_overlaps_nothing(written, other):
    """The last byte of `other` at the first byte of `written`, layer 2 on the written side, layer 0 (or 1) on the other."""
    c = stack()
    at = 1 << 45
    used = dict(q=2 * QH * 256, out=2 * QH * 512, hat=256 * 2 * D, workspace=4096)
    used |= {n: ((CAP + 128 if "raw" in n else (SINKS * 2 if "sink" in n else RECENT + 7)) * 2 * D) for n in READ if n[:3] in ("raw", "sin", "rec")}
    used |= {n: (CAP + 128) * (256 if "codes" in n else 16) for n in FIELDS}
    used |= {"staged_" + n: 256 * (256 if "codes" in n else 16) for n in FIELDS}
    if other == written:
        pytest.skip("one buffer")

    def put(name, where, l):
        if name == "workspace":
            c.workspace = where
        elif name[:3] == "hat":
            c.hat[int(name[3])] = where
        elif name[:4] == "rope":
            c.rope = tuple(where if i == int(name[4]) else x for i, x in enumerate(c.rope))
        else:
            setattr(c.layers[l], name, where)

    put(written, at, 2)
    size = used.get(other.rstrip("0123"), (SINKS + 128 + 7) * 256)          # rope: rows of the longest sequence
    put(other, at - size // 16 * 16 + 16, 1 if other[:3] == "raw" else 0)
    assert c.status() == B.AQUAKV_EINVAL, B.aquakv_last_error()
    assert "overlaps" in B.aquakv_last_error()


PARAMETERS = dict(w_k=D * D * 2, w_v=2 * D * D * 2, b_k=4 * D, b_v=4 * D, signs_k=D, signs_v=D, codebook=16 * 8,
                  search_table=B.aquakv_search_table_bytes(16))


@pytest.mark.parametrize("written", ["out", "staged_v_codes", "hat", "workspace"])
@pytest.mark.parametrize("name", PARAMETERS)
def test_nothing_is_written_over_the_parameters(name, written):
    """The last bytes of a layer's parameter at the first byte of a buffer that the call writes."""
    at = 1 << 45
    c = Call([layer(first=True), None, layer(**{name: at - PARAMETERS[name] // 16 * 16 + 16}), layer()])
    if written == "workspace":
        c.workspace = at
    elif written == "hat":
        c.hat[3] = at
    else:
        setattr(c.layers[0], written, at)
    assert c.status() == B.AQUAKV_EINVAL
    assert f"{name} of layer 2" in B.aquakv_last_error() and "overlaps" in B.aquakv_last_error()


@pytest.mark.parametrize("kw,want", [
    (dict(n_sink=[SINKS, SINKS + 1]), B.AQUAKV_EINVAL), (dict(n_compressed=[CAP + 1, 0]), B.AQUAKV_EINVAL),
    (dict(n_recent=[-1, 0]), B.AQUAKV_EINVAL), (dict(n_sink=[0, 4], n_compressed=[0, 128], n_recent=[0, 7]), B.AQUAKV_EINVAL),
    (dict(workspace_bytes=4096), B.AQUAKV_EWORKSPACE)])
def test_counts_and_workspace_of_a_cache_are_checked(kw, want):
    assert stack().status(**kw) == want


@pytest.mark.parametrize("name", WRITTEN + READ)
@pytest.mark.parametrize("value", [None, 1])
def test_every_buffer_of_a_cache_is_required_and_aligned(name, value):
    c = stack()
    entry = c.layers[1 if name[:3] == "raw" else 2]
    setattr(entry, name, None if value is None else getattr(entry, name) + 1)
    assert c.status() == (B.AQUAKV_ENULL if value is None else B.AQUAKV_EALIGN)


def test_copy_ranges_checks_its_list():
    B.aquakv_copy_ranges([])
    for bad in ([0, 1 << 40, 16], [1 << 40, 0, 16], [0, 0, 0, 1 << 40, 0, 1]):
        with pytest.raises(B.AquaKVError) as e:
            B.aquakv_copy_ranges(bad)
        assert e.value.status == B.AQUAKV_ENULL
