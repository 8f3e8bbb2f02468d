"""bench.py's rows of the velocity-OE and stage-map kernels on the CPU: the bytes that are reported are those of the
tables the kernels hold, and the hydro OE sensor has a row, counters and a share of the flops of its own."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


@pytest.mark.parametrize("N,k", [(1, 0), (2, 2), (3, 2), (4, 3), (5, 5), (6, 5)])
def test_velocity_oe_rows_count_the_table_that_is_held(N, k):
    import bench
    src = open(os.path.join(bench.CSRC, "common.h")).read()
    assert re.search(r"psi_modes\(int p\) \{ return p \* p; \}", src)  # the rows that the kernels write
    nn, row = (N + 1) ** 2, (N * N + 1) // 2 * 2
    t = {r[2]: r for r in bench.kernel_table(N, k)}
    assert bench.kernel_bytes(t["k_vel_prep<"], N) == nn * 8 + nn * row * 8
    assert bench.kernel_bytes(t["k_vel_proj<"], N) == nn * row * 8 + 9 * nn * 8 + (N + 1) * 8
    for r in t.values():
        assert 0.0 < r[6] <= 1.0, r[2]


def test_hydro_sensor_row():
    import bench
    t = {r[2]: r for r in bench.kernel_table(4, 3)}
    assert t["k_hydro_sensor<"][0] == 8 and t["k_hydro_oe_pp<"][0] == 1
    assert t["k_hydro_sensor<"][4] == 5 * 25 * 8 + 15 * 8 + 5 * 8
    assert t["k_hydro_sensor<"][5] + t["k_hydro_oe_pp<"][5] == bench.oe_pp_flops(1, 5)
    assert len({r[0] for r in t.values()}) == len(t)


@pytest.mark.gpu
@pytest.mark.parametrize("n,sensor", [(64, True), (16, False)])
def test_sensor_time_is_part_of_the_map(n, sensor):
    """Ids 1 and 8 of the kernel timing over more launches than the event pool holds."""
    import paper_2609_10849_amd as pk
    from paper_2609_10849_amd import workloads as W
    from tests._gpu import announce, dev
    announce("kernel timing %d" % n)
    L, U, *_ = W.isentropic_vortex(n, n, 3, 2)
    S = pk.Solver.from_layout(L, pk.Options.make(oe_hydro=1, pp=1))
    g = dev(U)
    S.timing(True)
    for _ in range(130):
        assert S.hydro_substep(g, 1e-4)[0] == 0
    S.timing(False)
    (a, ta), (b, tb), (c, tc) = (S.timing_read(i) for i in (0, 1, 8))
    S.close()
    assert a == b == 390 and c == (390 if sensor else 0)
    assert 0.0 < ta < 390 and 0.0 < tb < 390  # a launch takes microseconds
    assert (0.0 < tc < tb) if sensor else tc == 0.0
