"""Passes of 33 to 48 columns, which take three column tiles, through the solvers that pack and read their operands by columns."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,t", [(700, 34), (4097, 49), (9001, 48), (17000, 113)])
def test_cg_columns(n, t):
    from tests.test_gpu_cg_columns import test_iterates_follow_the_textbook_recurrence as follow
    follow(n, 5, "matern32", t)


@pytest.mark.parametrize("n,block,t", [(1025, 100, 40), (4097, 500, 113)])
def test_ap_columns(n, block, t):
    from tests.test_gpu_ap_columns import test_steps_follow_the_projection as follow
    follow(n, block, t, True)


@pytest.mark.parametrize("n,t,batch", [(2100, 34, 300), (4100, 49, 700), (9000, 112, 333)])
def test_sgd_columns(n, t, batch):
    from tests.test_gpu_sgd_columns import test_iterates_follow_the_step as follow
    follow(n, t, batch, "se")
