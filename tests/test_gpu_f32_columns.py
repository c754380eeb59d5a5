"""The binary32 slow model in one launch at the edges of its two forms: 4 and 16 rows a block (2,048 rows and one more on 256
compute units), one, two and four columns a lane (outputs around 16, 32, 64, 128, 256), inputs around whole groups of 16, weights
off the 16-byte grid.  The same check as test_gpu_f32_rows: logits bit for bit."""
import pytest

from test_gpu_f32_rows import test_rows as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,dims", [
    (2048, (16, 128, 129, 16)), (2049, (17, 128, 16, 17)), (2050, (48, 256, 257, 64)), (2051, (1, 65, 64, 33)), (4099, (65, 33, 32, 1)),
    (5, (129, 16, 17, 2)), (1023, (15, 1, 47, 10)), (40000, (12, 20, 24, 3)), (33, (1200, 1100, 60, 5))])
def test_forms(rows, dims):
    check(rows, dims, 0)
