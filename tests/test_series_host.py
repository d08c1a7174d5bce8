"""Where the one-launch series may run (host logic, no GPU): its workgroups wait for each
other, so the device has to hold all of them."""
import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_1203_6208_amd import rpy
    return rpy._lib


# (beads, adaptive, workgroups): 8 beads per workgroup to 512 for a fixed order, else 4
GROUPS = [(1, 0, 1), (100, 0, 13), (512, 0, 64), (513, 0, 129), (1000, 0, 250), (1024, 0, 256),
          (1, 1, 1), (100, 1, 25), (512, 1, 128), (513, 1, 129), (1024, 1, 256)]


@pytest.mark.parametrize("n,adaptive,groups", GROUPS)
def test_needs_every_workgroup_resident(lib, n, adaptive, groups):
    use = lib.rpy_host_series_use
    for per_cu in (1, 2, 3):
        for cus in (1, 16, 32, 64, 80, 128, 129, 256, 304):
            held = per_cu * cus
            assert use(n, adaptive, per_cu, cus) == (0 if held < groups else 1 if held < 4 * groups else 2)
    assert use(n, adaptive, 0, 256) == 0   # occupancy unknown


def test_full_device_and_partitions(lib):
    use = lib.rpy_host_series_use
    assert [use(n, 0, 1, 256) for n in (100, 512, 513, 1000, 1024, 1025)] == [2, 2, 1, 1, 1, 0]
    assert use(512, 1, 2, 256) == 2
    assert use(1000, 0, 1, 128) == 0 and use(1000, 0, 1, 32) == 0   # a part of the device
    assert use(512, 0, 1, 32) == 0 and use(256, 0, 1, 32) == 1 and use(64, 0, 1, 32) == 2
