"""The corrections of centred plans at the edges of their tiles: block counts around the
matrix cores' 16, sketches of one to seven column tiles, rows short of a vector, a tile
and a chunk. Against the oracle with the tolerances of the centred parity test."""

import pytest
import torch

from test_gpu_center import centred_case, field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ny,K,N,r,p", [
    (9, 7, 2, 20, 6, 4),        # fewer rows than a wave
    (41, 25, 16, 20, 20, 12),   # one row into a fifth tile
    (37, 29, 17, 20, 30, 11),   # one block past a group of 16
    (64, 51, 33, 12, 60, 10),
    (45, 45, 20, 20, 80, 10),
    (63, 65, 15, 24, 100, 12),  # widest sketch that leaves room for the indicators
])
def test_centred_tiles(nx, ny, K, N, r, p, dtype):
    St = field(nx, ny, K * N, N, seed=nx + K, n_modes=min(100, nx * ny // 2))
    centred_case(St, r, p, 1, 5, dtype, N, name="centred-tiles")
