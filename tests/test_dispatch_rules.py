"""The rules that choose between the forms of a kernel, at sizes where one form
was measured the faster by 4% or more on an MI355X (times in microseconds)."""
import pytest

from dispatch import rule


@pytest.mark.parametrize("rows,r,batch,narrow,wide", [
    (4096, 1024, 1, 45.3, 100.0), (4096, 1024, 4, 78.8, 147.3), (4096, 1024, 8, 116.8, 159.6),
    (4096, 1024, 10, 180.1, 170.7), (4096, 1024, 16, 255.9, 225.1), (4096, 1024, 64, 988.0, 663.0),
    (4096, 256, 32, 142.9, 181.4), (2048, 256, 1, 33.9, 58.6), (2048, 256, 32, 72.4, 85.7),
    (2048, 256, 64, 146.5, 114.1), (1024, 256, 1, 30.3, 37.1), (1024, 256, 48, 59.4, 53.3),
    (512, 128, 1, 29.4, 27.5), (512, 128, 64, 38.4, 29.9), (512, 32, 16, 29.1, 26.9)])
def test_sign_columns(rows, r, batch, narrow, wide):
    assert rule("narrow_sign_columns", rows, r, batch) == (narrow < wide)


@pytest.mark.parametrize("r,batch,narrow,wide", [
    (1024, 1, 19.0, 38.8), (1024, 8, 80.1, 67.4), (1024, 16, 162.0, 107.5), (1024, 64, 682.3, 363.6),
    (256, 32, 22.0, 18.5), (256, 64, 41.7, 20.5), (512, 16, 40.0, 34.3), (512, 64, 160.8, 90.4)])
def test_align_columns(r, batch, narrow, wide):
    assert rule("narrow_align_columns", r, batch) == (narrow < wide)
