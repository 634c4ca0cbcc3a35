"""The bfloat16 attention descriptor's kernels at the edges of their blocks and instances:
neighbour counts around multiples of 16 (odd counts of blocks too: one matrix instruction
takes two), the last count of the 12-wave instance (96) and the capacity (120).

Each cluster is computed alone (a workgroup of 8 waves per atom) and beside a far-away one
that takes the system past the size from which two atoms share 12 waves (lists over 96 go to
8 waves there too): the same bits.  Forces against the FP64 oracle, divided by the
oracle's largest: a force passes 13 rounded products forward (embedding, and Q, K, scores,
V, output of two layers) and as many backward, each operand off by up to 2^-9 of itself; added
up linearly over two operands, 2 * 26 * 2^-9 = 0.1."""
import numpy as np
import pytest

from oracle.dp import evaluate
from test_gpu_descriptor_tiles import _ball

pytestmark = pytest.mark.gpu

BOUND = 2 * 26 * 2.0 ** -9


@pytest.mark.parametrize("n", [2, 16, 17, 18, 33, 34, 81, 97, 98, 113, 114, 121])
def test_neighbour_counts_at_block_edges(gpu_bf16, omodel, n):
    X, t = _ball(n, 2.95, 0.8, 5)
    ref = evaluate(omodel, X, t, None)
    assert int(ref["nnei"].min()) == n - 1
    alone = gpu_bf16.compute(X, t, None, atom_energy=True)
    top = np.max(np.abs(ref["F"]))
    f = np.max(np.abs(alone["F"] - ref["F"])) / top
    print(n, "largest force", top, "error", f)
    assert f <= BOUND
    Y, u = _ball(257, 6.0, 1.0, 7)
    both = gpu_bf16.compute(np.concatenate([X, Y + 100.0]), np.concatenate([t, u]), None, atom_energy=True)
    assert np.array_equal(alone["E_i"], both["E_i"][:n]) and np.array_equal(alone["F"], both["F"][:n])
