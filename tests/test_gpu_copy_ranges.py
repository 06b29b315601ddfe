"""aquakv_copy_ranges: many byte ranges in one launch, against slicing on the host."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    (16,), (2,), (1, 3, 7), (16384, 16368, 16400), (0, 2048, 0), (5 << 20, 2048, 6), tuple(2048 + 16 * (i % 5) for i in range(131)),
    tuple(2 + 2 * (i % 9) for i in range(257))])
@pytest.mark.parametrize("shift", [0, 2, 1])
def test_copies_every_range_and_nothing_else(sizes, shift):
    from paper_2501_19392_amd import binding as B
    gen = torch.Generator().manual_seed(sum(sizes) + shift)
    src, want, jobs, at = [], None, [], 0
    total = sum(s + 64 for s in sizes) + 64
    dst = torch.full((total,), 7, dtype=torch.uint8, device="cuda")
    want = dst.cpu()
    for n in sizes:
        x = torch.randint(0, 256, (n + 32,), generator=gen, dtype=torch.uint8)
        src.append(x.cuda())
        d = (at + 15) // 16 * 16 + shift
        want[d:d + n] = x[shift:shift + n]
        jobs += (dst.data_ptr() + d, src[-1].data_ptr() + shift, n)
        at = d + n
    print(f"case copy_ranges {len(sizes)} ranges, shift {shift}", flush=True)
    B.aquakv_copy_ranges(jobs)
    torch.cuda.synchronize()
    assert torch.equal(dst.cpu(), want)


def test_rejects_null_pointers_before_any_launch():
    from paper_2501_19392_amd import binding as B
    B.aquakv_copy_ranges([])
    B.aquakv_copy_ranges([0, 0, 0])
    with pytest.raises(B.AquaKVError):
        B.aquakv_copy_ranges([0, 4096, 16])
