"""What the library launches for given sizes, without a GPU (see launches.py)."""
import os

import pytest

from paper_2403_07816_amd import binding as B

from launches import P, adamw_call, launches

MAX_THREADS = (1 << 32) - 1     # of one launch and direction of the grid


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if not os.path.exists(B.LIB_PATH):
        from paper_2403_07816_amd.build import build
        build(verbose=False)
    folder = tmp_path_factory.mktemp("launches")
    return lambda *calls: launches(list(calls), str(folder))


def threads_fit(launch):
    return all(g * b <= MAX_THREADS for g, b in zip(launch.grid, launch.block))


@pytest.mark.parametrize("dtype", [B.BTX_F32, B.BTX_BF16])
@pytest.mark.parametrize("n", [1, 4097, (1 << 34) - 1024, (1 << 34) + 5, 1 << 36])
def test_adamw_takes_tensors_of_any_length(record, n, dtype):
    """Every element belongs to one launch, in pieces of whole 16-byte chunks where one launch cannot hold the threads."""
    (rc, found), = record(adamw_call(n, dtype))
    assert rc == 0 and found
    done = 0
    for launch in found:
        assert threads_fit(launch)
        assert launch.first == P + 4 * done and done % 4 == 0       # the master weights of this piece
        done += launch.grid[0] * 1024                               # at most; the last workgroup may hold fewer
    assert done - 1024 < n <= done + 3                              # (up to 3 trailing elements go to the first workgroup)
