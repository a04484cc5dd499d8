"""How many key streams the bf16 attention kernels take (plan.cpp's rule, through the host
shim; CPU only), against times measured with each stream count on 256 CUs."""
import pytest

CUS = 256

# d, heads, groups a head, rows a group, {tiles: us with 1, 2 (, 4) streams}
MEASURED = [
    (128, 5, 3, 1560, {1: (12.6, 13.5), 2: (14.1, 13.1), 8: (22.1, 17.9), 32: (54.9, 35.9), 64: (98.1, 59.9)}),
    (128, 12, 1, 4680, {1: (13.5, 24.9), 8: (23.9, 33.7), 64: (111.3, 123.2)}),
    (128, 40, 3, 1560, {1: (46.8, 79.7), 8: (85.6, 109.2), 16: (131.4, 155.5), 32: (226.0, 245.7), 64: (415.7, 429.5)}),
    (128, 16, 1, 4680, {4: (32.2, 38.6), 8: (43.6, 48.5), 32: (115.1, 107.0), 64: (210.8, 184.7)}),
    (128, 12, 73, 64, {1: (40.3, 45.7), 4: (56.3, 50.3), 64: (364.2, 215.3)}),
    (64, 16, 1, 1560, {1: (7.4, 8.3, 14.6), 4: (11.0, 9.2, 14.1), 16: (25.1, 16.5, 21.8), 64: (81.6, 43.5, 52.7)}),
    (64, 40, 1, 1560, {1: (11.4, 17.7, 27.0), 4: (17.9, 20.5, 26.1), 16: (41.9, 41.1, 41.7), 64: (139.2, 127.8, 106.4)}),
    (64, 16, 1, 4680, {1: (12.9, 19.6, 32.8), 4: (20.3, 22.3, 31.9), 16: (48.9, 43.1, 50.9), 64: (165.4, 130.7, 131.6)}),
    (64, 12, 1, 4680, {1: (8.0, 14.0, 26.8), 4: (11.8, 15.9, 26.0), 64: (83.4, 86.8, 105.8)}),
    (64, 12, 73, 64, {1: (18.5, 23.2, 27.3), 4: (29.5, 27.3, 27.2), 64: (233.4, 159.5, 106.6)}),
    (64, 40, 3, 1560, {1: (23.7, 42.4, 78.3), 4: (37.3, 48.9, 76.2), 16: (89.6, 95.9, 121.9), 64: (300.5, 298.3, 313.1)}),
]


@pytest.mark.parametrize("d,H,R,rows,times", MEASURED)
def test_choice_against_times(host_shim, d, H, R, rows, times):
    for tiles, us in times.items():
        chosen = us[(1, 2, 4).index(host_shim.shim_key_streams(d, H * R, rows, tiles, CUS))]
        assert chosen <= 1.02 * min(us), (tiles, us, chosen)


def test_one_tile_takes_one_stream(host_shim):
    for d in (64, 128):
        for groups in (1, 7, 120, 4000):
            for rows in (33, 64, 65, 128, 300, 4680):
                for tiles in (0, 1):
                    assert host_shim.shim_key_streams(d, groups, rows, tiles, CUS) == 1, (d, groups, rows, tiles)
