"""FP64 wide rows on both sides of the line between whole rows and slabs in
the edge stage (256 points, 1.5 million point-features, 16-feature slabs up to
512 points), against the oracle's trajectory: 1e-11 relative."""
import pytest

from tests.test_gpu_wide import follow, problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


@pytest.mark.parametrize("n,p", [(255, 5890), (256, 5856), (256, 5857), (512, 2932), (513, 2932)])
def test_both_sides_of_the_line(cc, n, p):
    follow(cc, *problem(n, p, 4, n % 2 == 0), "f64", 3.0, 6, 1e-11)
