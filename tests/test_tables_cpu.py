"""The library's sampling tables against the oracle's, entry for entry, over the
distributions a spec may name: whole-number tables have no tolerance."""
import math

import numpy as np
import pytest

import workloads as W


@pytest.fixture(scope="module")
def cxm():
    from paper_2507_01522_amd import cx
    return cx


# narrow and wide stays (each entry its own erfc call; one series over many), stays
# of less than a step and of many tables' length, tables of one entry to the longest
DWELLS = [(mu, sg, n) for mu in (-30.0, 0.0, math.log(36.0), 6.5, 40.0)
          for sg, n in ((1e-3, 300), (0.05, 1024), (0.5, 1024), (0.5, 4096), (3.0, 4096), (50.0, 77), (1e6, 4096))]
DWELLS += [(math.log(12.0), 0.4, n) for n in (1, 2, 3, 4, 5, 6, 255, 256, 257)]


@pytest.mark.parametrize("mu,sigma,n", DWELLS)
def test_dwell_tables(cxm, oracle_lib, mu, sigma, n):
    spec = W.tiny_parity_station().replace(dwell_mu=mu, dwell_sigma=sigma, dwell_max=n)
    td = cxm.build_tables(spec)[1]
    assert np.array_equal(td[1:], oracle_lib.OracleClass(spec).tables()[1][1:])


@pytest.mark.parametrize("seed", range(8))
def test_dwell_tables_drawn(cxm, oracle_lib, seed):
    rng = np.random.default_rng(seed)
    for _ in range(25):
        spec = W.tiny_parity_station().replace(dwell_mu=float(rng.uniform(-2, 8)),
                                               dwell_sigma=float(10 ** rng.uniform(-2, 1)), dwell_max=4096)
        td = cxm.build_tables(spec)[1]
        assert np.array_equal(td[1:], oracle_lib.OracleClass(spec).tables()[1][1:])


@pytest.mark.parametrize("steps", [1, 7, 8, 9, 96, 288])
@pytest.mark.parametrize("peak", [0.0, 1e-12, 0.3, 2.5, 8.0])
def test_arrival_tables(cxm, oracle_lib, steps, peak):
    rng = np.random.default_rng(steps)
    base = W.tiny_parity_station().replace(steps_per_episode=steps, arrival_peak=peak)
    for spec in (base, base.replace(arrival_rate=rng.uniform(0.0, max(peak, 1e-9), steps))):
        assert np.array_equal(cxm.build_tables(spec)[0], oracle_lib.OracleClass(spec).tables()[0])
