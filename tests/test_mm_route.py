"""Which kernel a matmul takes (no GPU needed): the rule is a function of the
sizes, evaluated on the host."""
import pytest

import mm_routes as R

# Products timed on MI355X in the small tiles and in the 256 x 256 kernel (us).
SLOWER_IN_SMALL_TILES = {(717, 2304, 768): (8.6, 8.1), (555, 4096, 4096): (26.4, 25.3), (768, 4096, 4096): (26.9, 25.6),
                         (1024, 4096, 4096): (27.8, 26.4), (256, 12288, 4096): (28.3, 27.6), (100, 22016, 4096): (33.8, 30.7),
                         (768, 2816, 1024): (10.3, 9.2), (450, 8192, 4096): (28.0, 26.2), (256, 11008, 4096): (26.9, 25.5)}
FASTER_IN_SMALL_TILES = {(33, 768, 768): (3.4, 6.8), (64, 4096, 11008): (16.8, 55.8), (301, 4096, 4096): (15.6, 20.9),
                         (512, 8192, 8192): (45.5, 48.3), (1024, 768, 768): (6.0, 7.8), (1024, 512, 512): (4.6, 6.6),
                         (1000, 4096, 11008): (57.0, 67.1), (512, 1024, 8192): (17.5, 46.1)}


@pytest.mark.parametrize("shape", SLOWER_IN_SMALL_TILES, ids=str)
def test_products_slower_in_small_tiles_take_large_ones(shape):
    assert R.kernel(*shape) == R.MAIN


@pytest.mark.parametrize("shape", FASTER_IN_SMALL_TILES, ids=str)
def test_products_faster_in_small_tiles_take_them(shape):
    assert R.kernel(*shape) == R.STREAM


def test_rows_of_a_decode_and_odd_contractions():
    assert all(R.kernel(m, n, 4096) == R.STREAM for m in (1, 16, 32) for n in (64, 4096, 57344))
    assert all(R.kernel(512, 4096, k) == R.RAGGED for k in (1, 127, 4032, 4097, 1 << 22))


def test_amax_changes_the_tile_but_not_the_order_of_the_sums():
    """Each workgroup's fold of its maximum waits for the others', so calls that
    take the amax use fewer, larger tiles, of the same stage length."""
    for m in (1, 16, 33, 64, 100, 160, 256, 400, 717, 1024, 1531, 2048):
        for n in (512, 768, 1024, 2304, 4096, 12288):
            for k in (128, 512, 768, 1024, 3072, 4096):
                (kp, *tp), (ka, *ta) = R.route(m, n, k), R.route(m, n, k, with_amax=True)
                assert kp == ka, (m, n, k)
                if kp == R.STREAM:
                    assert R.stage(*tp) == R.stage(*ta), (m, n, k)
                    assert R.workgroups(m, n, *ta) <= R.workgroups(m, n, *tp), (m, n, k)
    # with the tile that is best without an amax: 22, 17.8 and 25 us with an in-launch bias
    for (m, n, k), most in {(256, 768, 768): 150, (64, 3072, 768): 200, (33, 4096, 4096): 256}.items():
        assert R.workgroups(m, n, *R.route(m, n, k, with_amax=True)[1:]) <= most


def test_wide_weights_of_short_rows_take_wide_tiles():
    """One token through a weight of many short rows: rounds of small
    workgroups cost more than their copies.  us in 32- or 48-column tiles, and
    in the widest: 9.8 and 6.7, 7.1 and 5.4, 13.3 and 11.2.
    Long rows keep what they had."""
    for n, k in ((57344, 128), (22016, 768), (57344, 768)):
        assert R.workgroups(1, n, *R.route(1, n, k)[1:]) <= 512, (n, k)
    assert R.route(1, 22016, 4096)[1:] == (1, 3) and R.route(16, 57344, 8192)[1:] == (1, 2)
