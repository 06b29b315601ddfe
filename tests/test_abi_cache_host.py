"""Host-side checks of the calls of the cache manager (aquakv_attend_cache, aquakv_copy_ranges): bad arguments are refused before the
device is touched.  No GPU needed: the addresses are made up and never dereferenced."""
import pytest

from paper_2501_19392_amd import binding as B

MiB = 1 << 20
H, QH, D = 8, 32, 1024
CAP, SINKS, RECENT = 256, 4, 128
FIELDS = ("k_codes", "k_scales", "v_codes", "v_scales")


def layer(first=False, **kw):
    base = 0x10000                                        # parameters: never compared, never read here
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
