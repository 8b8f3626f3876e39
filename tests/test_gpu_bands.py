"""Products whose tiles are walked in bands of four or eight tile rows: every tile once, at last bands of one row to a whole one, on both sides of the lines."""
import pytest

from test_gpu_parity import check_step

pytestmark = pytest.mark.gpu

# frames, D, H; tile height of the input product, its tile rows, rows of a band.  Single frames: as many rows as sequences.  (test_dispatch_cpu.py checks the tiles.)
BANDS = [
    (257, 24, 40, 64, 5, 4), (320, 24, 40, 64, 5, 4), (321, 24, 40, 64, 6, 4), (576, 24, 40, 64, 9, 4),   # bands of four: a last one of one row, ragged and whole, of two
    (2048, 24, 40, 64, 32, 4), (2049, 24, 40, 64, 33, 4), (2112, 24, 40, 64, 33, 4), (2560, 24, 40, 64, 40, 4), (2561, 24, 40, 64, 41, 4),
    (4224, 2048, 264, 128, 33, 4), (4097, 2048, 264, 128, 33, 4),
    (8192, 24, 40, 128, 64, 4), (8193, 24, 40, 128, 65, 4),  # at the line of the input gradients, of which a last band of eight has one row
    (16384, 24, 40, 128, 128, 4),                            # at the line of the input products
    (16385, 24, 40, 128, 129, 8), (16512, 24, 40, 128, 129, 8), (17409, 24, 40, 128, 137, 8),   # bands of eight: a last one of one row
]


@pytest.mark.parametrize("M,D,H,height,rows,band", BANDS)
def test_bands_of_tile_rows(M, D, H, height, rows, band):
    # From 8192 frames on with larger weights and eight classes: with small ones dz is nearly the same for all frames of a label and is rounded to bf16 alike, which leaves up to
    # 0.0252 (8192 frames, 150 classes) of the lower layer's bias gradient, a sum that nearly cancels; float64 with that rounding gives the same number.  So it leaves 0.0017 at most.
    many = M >= 8192
    check_step(dict(T=1, B=M, D=D, H=H, L=1 if D > 24 else 2, P=0, V=8 if D > 24 or many else 150), 1, seed=97, theta_scale=3.0 if many else 1.0)


@pytest.mark.parametrize("T,B,H", [
    (3, 40, 576), (3, 40, 616), (3, 40, 640), (2, 60, 704), (3, 40, 768), (3, 40, 776),   # weight gradients of 9, 10 (ragged and whole), 11, 12 and 13 tile rows, of 3 to 13 columns
])
def test_bands_of_weight_gradients(T, B, H):
    check_step(dict(T=T, B=B, D=264, H=H, L=2, P=0, V=20), 1, seed=97)


@pytest.mark.parametrize("T,B", [
    (5, 128), (7, 128), (2, 500),                # products on 64-row tiles: 10, 14 and 16 tile rows, bands of four
    (32, 128), (33, 128), (34, 125), (41, 128),  # 64, 66, 67 and 82
    (33, 256),                                   # on 128-row tiles: 66
])
def test_bands(T, B):
    # 32 x 128: the bias gradient nearly cancels over the frames, and bf16's rounding of dE/da alone leaves 0.026855 of its largest
    # element, digit for digit also where all bands have eight rows; a tile left out or taken twice is 1/32 of the rows, error near 1
    check_step(dict(T=T, B=B, D=24, H=40, L=2, P=0, V=150), 1, seed=97, theta_scale=1.0, tol=0.03 if (T, B) == (32, 128) else None)
