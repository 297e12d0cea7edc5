"""The byte model of bench.py's roofline figures."""
import bench


def test_the_preprocess_backward_is_charged_for_the_splats_it_reads():
    """Heavy overlap at 1920x1080: 5M splats, nearly all of them listed, a tenth with a row of the backward raster.  Every
    splat has a visibility word in and 59 gradients out, a splat with a row its 59 parameters and 10 binary64 sums in;
    a listed splat without a row is not read."""
    n, listed, rows = 5_000_000, 4_900_000, 480_000
    floats = 3 + 3 + 4 + 1 + 1 + 48
    want = n * (4 + 4 * floats) + rows * (4 * floats + 80)
    for L in (listed, listed // 2):
        assert bench.algorithmic_bytes("preprocess_backward", n, 16, 0, 0, L, 1920 * 1080, R=rows, S=rows) == want
        # with the update fused in, a parameter and its two moments in and out instead
        assert bench.algorithmic_bytes("preprocess_backward_adam", n, 16, 0, 0, L, 1920 * 1080, S=rows) == \
            n * (4 + 24 * floats) + rows * 80
