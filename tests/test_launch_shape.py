"""The launch shape of a thread is what its reader reports: setting that again restores
the state, also the one in which no shape is set and each kernel chooses its own."""
import threading

import pytest


@pytest.fixture()
def A():
    from paper_2012_14332_amd import abc
    keep = abc.get_launch_config()
    yield abc
    abc.set_launch_config(*keep)


def test_no_shape_reads_as_zeros_and_is_restored(A):
    A.set_launch_config(0, 0, 0)
    assert A.get_launch_config() == (0, 0, 0)
    keep = A.get_launch_config()
    A.set_launch_config(2, 256, 3)
    A.set_launch_config(*keep)
    assert A.get_launch_config() == (0, 0, 0)


@pytest.mark.parametrize("shape,read", [((1, 512, 2), (1, 512, 2)), ((4, 0, 0), (4, 128, 2)), ((0, 0, 3), (1, 512, 3))])
def test_a_shape_is_read_and_written_back(A, shape, read):
    A.set_launch_config(*shape)
    assert A.get_launch_config() == read
    A.set_launch_config(*A.get_launch_config())
    assert A.get_launch_config() == read


def test_the_shape_belongs_to_the_thread(A):
    A.set_launch_config(1, 256, 2)
    seen = []
    t = threading.Thread(target=lambda: seen.append(A.get_launch_config()))
    t.start()
    t.join()
    assert seen == [(0, 0, 0)] and A.get_launch_config() == (1, 256, 2)
