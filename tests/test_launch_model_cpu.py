"""Which launches the host code makes, on the fake HIP device under
AddressSanitizer + UndefinedBehaviorSanitizer: tests/sanitize/drive_launches.cpp
makes the calls, the fake device checks every range their launches would touch,
and that no graph is destroyed while a launch of it is in flight."""
import pytest

from tests.sanitize import build as SB
from tests.test_host_sanitizers_cpu import run


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return SB.build("asan", str(tmp_path_factory.mktemp("launches")), "drive_launches")


@pytest.mark.parametrize("section", ["horizons", "parts", "stage", "policy", "grids"])
def test_launches(driver, section):
    rc, out = run([driver, section], {"ASAN_OPTIONS": "detect_leaks=1"})
    assert rc == 0 and "DRIVE OK" in out, out[-4000:]
    assert "graph execs destroyed with launches in flight: 0" in out
    assert "device allocations left: 0" in out
