"""Host-side logic of the GPU parity tests, checked without a GPU."""
import numpy as np
import pytest

import torch

from paper_2510_10129_amd import _lib
from test_gpu_layer import _stratified_rows


@pytest.mark.parametrize("M,g", [(1, 1), (64, 4), (883, 4), (3404, 4), (16576, 4), (14539, 7), (13363, 8), (500, 1),
                                 (700, 2), (257, 32)])
def test_stratified_rows_cover_every_attention_block_and_gemm_tile(M, g):
    rows = _stratified_rows(M, g, 16, seed=M + g)
    assert rows[0] == 0 and rows[-1] == M - 1 and np.all(np.diff(rows) > 0) and rows.max() < M
    cols = set()
    for r in rows:                                   # the 256-column blocks of (token, head) columns a row touches
        cols.update(range((r * g) // 256, (r * g + g - 1) // 256 + 1))
    assert cols >= set(range((M * g + 255) // 256))
    for tile in (128, 192, 256):                     # every row tile of these heights holds a compared row
        assert set(rows // tile) == set(range((M + tile - 1) // tile)), tile


@pytest.mark.parametrize("kind", [int, np.int64, np.int32, np.uint32, np.uint8, np.int16, bool])
def test_block_descriptors_take_any_integer(kind):
    """Column and length of a batched tensor's block come through as they are, whatever integer type a caller keeps them in."""
    a = torch.zeros(2, 3, 60)[:, :, 4:]                      # strides of a view
    arr, H, Q_a = _lib.Context._aux_blocks([(a, kind(1), kind(1)), (a, 2, kind(1)), (a, kind(0), 54)])
    assert (H, Q_a) == (2, 3) and [(b.col0, b.len) for b in arr] == [(1, 1), (2, 1), (0, 54)]
    assert all((b.attn, b.stride_head, b.stride_row) == (a.data_ptr(), 180, 60) for b in arr)


def test_block_descriptors_refuse_what_is_no_integer():
    a = torch.zeros(2, 3, 60)
    for blocks in ([(a, 2.0, 40)], [(a, 2, 40.0)], [(a, -1 << 40, 4)]):
        with pytest.raises(TypeError):
            _lib.Context._aux_blocks(blocks)
    for blocks in ([(a, 30, 31)], [(a[0], 2, 40)], [(a.transpose(1, 2), 0, 2)], [(a, 2, 40), (a[:1], 2, 40)]):
        with pytest.raises(ValueError):
            _lib.Context._aux_blocks(blocks)


@pytest.mark.parametrize("kind", [int, np.int64, np.int32, np.uint8])
def test_chunk_descriptors_take_any_integer_prefix(kind):
    """The chunk table of a cache assembly: own rows of every chunk behind a prefix in any integer type."""
    chunks = [torch.zeros(n, 2, 64, dtype=torch.bfloat16) for n in (16, 7, 300)]
    dst = _lib.KVLayer(torch.zeros(400, 2, 64, dtype=torch.bfloat16), torch.zeros(400, 2, 64, dtype=torch.bfloat16))
    seen = {}

    class Lib:
        def cc_assemble_cache(self, h, arr, n, P, st, sh, n_tail, kv):
            seen.update(table=[(c.K, c.V, c.len) for c in arr], args=(n, int(P), st, sh, n_tail))
            return _lib.CC_OK

    ctx = _lib.Context.__new__(_lib.Context)
    ctx._lib, ctx._h = Lib(), None
    ctx.assemble_cache(chunks, chunks, kind(5), 3, dst)
    assert seen["table"] == [(c.data_ptr(), c.data_ptr(), len(c) - 5) for c in chunks] and seen["args"] == (3, 5, 128, 64, 3)
