"""dgc_permute_records against torch indexing: every piece width (16, 8 and 4
bytes, chosen by the record size and the buffers' alignment), sizes around a
work-group's share, ids out of range left alone."""
from __future__ import annotations

import ctypes as C

import pytest

dgc = pytest.importorskip("paper_1601_07613_amd")
from paper_1601_07613_amd import _lib  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [1, 2, 3, 4, 5, 12, 18, 48, 84])
@pytest.mark.parametrize("off_src,off_dst", [(0, 0), (1, 0), (0, 2), (2, 2)])
@pytest.mark.parametrize("n", [1, 85, 341, 1024, 1025])
def test_permute_matches_indexing(gpu_device, words, off_src, off_dst, n):
    import torch

    g = torch.Generator().manual_seed(n * 100 + words)
    perm = torch.randperm(n, generator=g).int()
    if n > 4:
        perm[2], perm[3] = -1, n      # out of range: those records stay as they are
    ok = (perm >= 0) & (perm < n)
    src = torch.randint(-2**31, 2**31 - 1, (n * words + 4,), generator=g, dtype=torch.int64).int()
    S = src[off_src:off_src + n * words].view(n, words)
    d, p = src.cuda(), perm.cuda()
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    for to_layout in (1, 0):
        ref = torch.full((n, words), 7, dtype=torch.int32)
        if to_layout:
            ref[perm[ok].long()] = S[ok]
        else:
            ref[ok] = S[perm[ok].long()]
        out = torch.full((n * words + 8,), 7, dtype=torch.int32, device="cuda")
        _lib.check(_lib.load().dgc_permute_records(d.data_ptr() + 4 * off_src, out.data_ptr() + 4 * off_dst,
                                                   p.data_ptr(), n, 4 * words, to_layout, st), "permute")
        got = out.cpu()
        assert torch.equal(got[off_dst:off_dst + n * words].view(n, words), ref)
        assert (got[:off_dst] == 7).all() and (got[off_dst + n * words:] == 7).all()


# 12 pieces of 16, 9 of 8 and 5 of 4 bytes a record: the last call of one piece
# per work-item (at most 524,288 pieces), the first of four, and one beyond
@pytest.mark.parametrize("words,n", [(48, 43690), (48, 43691), (48, 60001), (18, 58254), (18, 58255), (5, 104857),
                                     (5, 104858)])
def test_permute_pieces_per_work_item(gpu_device, words, n):
    test_permute_matches_indexing(gpu_device, words, 0, 0, n)
