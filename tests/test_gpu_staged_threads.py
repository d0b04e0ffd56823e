"""moc_eval_batch_staged on either side of the sizes at which it takes more threads or more nodes a lane (768 candidates
among them), with few and with many further copies in a wave (one of a lane's is taken together with the other lanes', the rest one by one)."""
import pytest

from test_gpu_staged import moc, test_staged_recomputed_starts_and_ends as check  # noqa: F401  (moc: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,C,degree,B", [
    (64, 2, 2, 70), (65, 4, 6, 70), (128, 2, 3, 70), (129, 3, 2, 70), (256, 3, 5, 40), (257, 2, 3, 40), (1023, 4, 2, 20), (1024, 2, 5, 20),
    (64, 4, 3, 800), (65, 2, 2, 800), (128, 3, 6, 800), (129, 4, 2, 769), (256, 1, 3, 800), (257, 2, 2, 800), (512, 3, 3, 770), (512, 2, 2, 70),
    (1025, 2, 2, 20), (2047, 3, 3, 10), (2048, 1, 5, 10), (2049, 2, 3, 10), (2049, 1, 2, 10), (2049, 3, 2, 6), (4095, 2, 6, 5)])
def test_staged_thread_counts(moc, n, C, degree, B):  # noqa: F811
    check(moc, n, C, degree, B)
