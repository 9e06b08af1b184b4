"""The backward of float32 tensors with heads in eights, whose work-groups are dealt to the XCDs head by head, and with one head
less or more: every head's rows must come from its own work-groups."""
import pytest

import tests.test_backward_tiles_gpu as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L,u", [
    (1, 7, 130, 40), (1, 8, 130, 40), (3, 3, 130, 40), (2, 8, 40, 20),   # one or two groups of queries, blocks of 32 keys
    (6, 4, 700, 70), (5, 5, 700, 70),                                    # key splits and their partial sums
    (1, 8, 1700, 850), (1, 9, 1700, 850),                                # dQ from a kernel of its own
])
def test_heads_in_eights(B, H, L, u):
    tiles.test_tiles("f32", B, H, L, u)
