"""The coalesce's paths by batch size, at the edges of their tiles, against the oracle: every kernel
variant of the small batches (512, 1024 and 2048 tokens) with whole, partial and looped column
slices, vector and scalar rows, and both gradient types."""
import pytest

from test_gpu_by_owner import check_by_owner, grads_for, ids_for, owners

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 511, 512, 513, 1024, 1025, 2047, 2048])
@pytest.mark.parametrize("D,bf16", [(4, False), (36, False), (33, False), (260, True), (31, True)])
def test_small_batches(T, D, bf16):
    V, P = 700, 3
    ids = ids_for("zipf", T + D, T, V)
    ids[T // 2::97] = V + 1  # some tokens take no part
    check_by_owner(ids, grads_for(T * D, T, D, 0.01, bf16=bf16), V, owners("mod", V, P), P, bf16=bf16)


@pytest.mark.parametrize("T,D", [(2048, 4100), (1024, 2053), (300, 8196)])
def test_small_batches_of_wide_rows(T, D):
    # more column slices than one per XCD; a last slice that is not whole; a hot row
    V, P = 5000, 8
    ids = ids_for("zipf", T + D, T, V, 1.3)
    check_by_owner(ids, grads_for(T + D, T, D, 0.01), V, owners("range", V, P), P)
