"""GPU parity of the streaming projection kernel at the edges of its dispatch: one to eight row tiles (row shares from
seven on), k ranges of an odd number of k-tiles (half-empty pairs of narrow weights), n-tile counts that no workgroup
width divides, outputs narrow enough for a split along K."""
import pytest

import workloads as wl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "bf16w8", "bf16w4"])
@pytest.mark.parametrize("N,gamma", [(1, 1), (2, 8), (3, 6), (7, 7), (10, 8), (13, 8)])
def test_row_tiles_and_odd_k_ranges(N, gamma, dtype):
    """1, 16, 18, 49, 80 and 104 rows; three, six and five k-tiles."""
    w = wl.get_workload("c3").scaled(n_layers=2, d_model=96, n_heads=3, head_dim=64, d_ff=160, vocab=1008, N=N, gamma=gamma,
                                     S=70, R=9, seed=1300 + N, dtype=dtype)
    Case(w, branches=sorted({0, N // 2, N - 1})).run_oracle().run_gpu().compare()


@pytest.mark.parametrize("dtype", ["bf16", "bf16w8", "bf16w4"])
@pytest.mark.parametrize("N,gamma", [(2, 4), (4, 8), (6, 8)])
def test_split_k_with_ragged_splits(N, gamma, dtype):
    """8, 32 and 48 rows; the down projection has 169 k-tiles for 32 n-tiles, so it is split along K unevenly."""
    w = wl.get_workload("c3").scaled(n_layers=2, d_model=512, n_heads=4, head_dim=128, d_ff=5408, vocab=2000, N=N, gamma=gamma,
                                     S=64, R=5, seed=1400 + N, dtype=dtype)
    Case(w, branches=[0, N - 1]).run_oracle().run_gpu().compare()
