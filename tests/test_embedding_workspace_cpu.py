"""Workspace sizes of the embedding: a caller may keep a workspace sized once,
so the bytes asked for stay what they were."""

import pytest

from paper_2010_14058_amd import _lib


@pytest.mark.parametrize("n,nnz,dim,nbytes", [(600, 359_400, 16, 13_724_416),
                                              (2_000, 60_000, 4, 6_094_080),
                                              (20_000, 400_000, 16, 91_535_104),
                                              (20_000, 400_000, 256, 244_341_504),
                                              (1_000_000, 20_000_000, 128, 11_166_519_552)])
def test_bytes(n, nnz, dim, nbytes):
    assert _lib.load().tg_embedding_workspace_bytes(n, nnz, dim) == nbytes
