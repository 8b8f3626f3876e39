"""Products whose tiles are walked in bands of four or eight tile rows: every tile once, at last bands of one row to a whole one, on both sides of the lines."""
import pytest

from test_gpu_parity import check_step

pytestmark = pytest.mark.gpu

# frames, D, H; tile height of the input product, its tile rows, rows of a band.  Single frames: as many rows as sequences.  (test_dispatch_cpu.py checks the tiles.)
BANDS = [
    (257, 24, 40, 64, 5, 4), (320, 24, 40, 64, 5, 4), (321, 24, 40, 64, 6, 4), (576, 24, 40, 64, 9, 4),   # bands of four: a last one of one row, ragged and whole, of two
    (2048, 24, 40, 64, 32, 4),                               # at the line of 32 tile rows
    (2049, 24, 40, 64, 33, 8), (2112, 24, 40, 64, 33, 8), (2560, 24, 40, 64, 40, 8), (2561, 24, 40, 64, 41, 8),   # bands of eight: a last one of one row, whole bands
    (4224, 2048, 264, 128, 33, 4), (4097, 2048, 264, 128, 33, 4),   # beyond the line of 4 MB: four again, a last one of one row; the weight gradients have nine tile rows
]


@pytest.mark.parametrize("M,D,H,height,rows,band", BANDS)
def test_bands_of_tile_rows(M, D, H, height, rows, band):
    check_step(dict(T=1, B=M, D=D, H=H, L=1 if D > 24 else 2, P=0, V=8 if D > 24 else 150), 1, seed=97)


@pytest.mark.parametrize("T,B", [
    (5, 128), (7, 128), (2, 500),                # products on 64-row tiles: 10, 14 and 16 tile rows, bands of four
    (32, 128), (33, 128), (34, 125), (41, 128),  # 64, 66, 67 and 82, bands of eight
    (33, 256),                                   # on 128-row tiles: 66
])
def test_bands(T, B):
    # 32 x 128: the bias gradient nearly cancels over the frames, and bf16's rounding of dE/da alone leaves 0.026855 of its largest
    # element, digit for digit also where all bands have eight rows; a tile left out or taken twice is 1/32 of the rows, error near 1
    check_step(dict(T=T, B=B, D=24, H=40, L=2, P=0, V=150), 1, seed=97, theta_scale=1.0, tol=0.03 if (T, B) == (32, 128) else None)
