"""Gradients of narrow projections over more workgroups than wide ones take: batches
for which every workgroup of the limit runs, with an uneven last round.  Bars and
reasons are those of the edge cases."""
import pytest

import test_gpu_fno_cubes as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,batch", [(32, 65), (64, 33)])
def test_narrow_projection(hidden, batch):
    C.test_forward_and_gradients_at_the_edges(16, 1, hidden, 1, 3, 6, batch)
