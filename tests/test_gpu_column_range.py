"""The byte-table sweep stores only the columns of a layer between the first reachable one and the
one from which all its rows are constant (the memory of the best plans without a limit); readers
clamp.  These cases put both ends at tile and sample edges: everything saturated at once, nothing
reachable, zero memories, equal costs (the lowest index has to win on both sides of the end), and
budgets that end inside, at and just behind a tile.  Whole tables are compared with the oracle's."""
import numpy as np
import pytest

from paper_2211_13878_amd import binding, workloads
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu
PACK, PEEK, NO_PEEK, WIDE = (binding.GALV_DP_FORCE_PACK, binding.GALV_DP_FORCE_PEEK, binding.GALV_DP_NO_PEEK,
                             binding.GALV_DP_FORCE_WIDE_TILES)


@pytest.mark.parametrize("S", [1, 8, 16, 22, 44, 64, 128, 256])
@pytest.mark.parametrize("m_range", [(0, 0), (0, 3), (64, 64), (100, 400), (0, 900)])
def test_ends_of_the_stored_columns(S, m_range):
    L, E = 5, 1100
    for c_range, r_range in (((0, 2), (0, 1)), ((0, 1000), (0, 90)), ((10 ** 11, 10 ** 12), (0, 1000))):
        w = workloads.random_workload(7 * S + m_range[1], 4, L, S, E, nR=2, m_range=m_range, c_range=c_range,
                                      r_range=r_range, infeasible=0.1, zero_diagonal=False)
        w.budget[:] = (E, 255, 256, min(E, 3 * m_range[1] // 2))
        for flags in (PACK | PEEK, PACK | NO_PEEK, PACK | PEEK | WIDE):
            check_against_oracle(w, flags=flags, table_instances=[0, 1, 2, 3], allow_vacuous=S == 1)   # (one strategy: no plan where a layer is unusable)


@pytest.mark.parametrize("S", [9, 44, 200])
def test_two_layers_and_one_handle_after_another_instance_mix(S):
    """Two layers (nothing is computed ahead), then a handle whose instances change what they store
    between solves."""
    w = workloads.random_workload(S, 3, 2, S, 700, nR=1, m_range=(0, 300), c_range=(0, 50), r_range=(0, 20),
                                  infeasible=0.2, zero_diagonal=False)
    check_against_oracle(w, flags=PACK | PEEK, table_instances=[0, 1, 2])
    tight, loose = (workloads.random_workload(S + q, 3, 6, S, 700, nR=1, m_range=(0, hi), c_range=(0, 50),
                                              r_range=(0, 20), infeasible=0.1, zero_diagonal=False)
                    for q, hi in ((1, 20), (2, 350)))
    sol = binding.Solver(3, 6, S, 700, 1, PACK | PEEK)
    import oracle
    for w in (tight, loose, tight):
        cost, _ = sol.solve(*binding.upload(w))
        plan = sol.backtrack().cpu().numpy()
        for b, ref in enumerate(oracle.solve_workload(w, threads=4)):
            assert int(cost[b]) == ref.best_cost and (plan[b] == np.asarray(ref.plan)).all()
    sol.close()


@pytest.mark.parametrize("S", [6, 22, 128])
def test_one_batch_with_and_without_the_byte_table(S):
    """Instances on 64-bit integers keep 32-bit back-pointers beside the bytes of the others."""
    w = workloads.random_workload(S, 6, 5, S, 900, nR=2, m_range=(0, 200), c_range=(0, 5000), r_range=(0, 300),
                                  infeasible=0.05, zero_diagonal=False)
    w.c[::2] += 1 << 58
    w.R[::2] += 1 << 50
    w.budget[:] = 900
    _, _, _, status = check_against_oracle(w, flags=PACK | PEEK, table_instances=range(6))
    assert (status[::2] == binding.GALV_INSTANCE_OK_INT64).all() and (status[1::2] == binding.GALV_INSTANCE_OK_FAST_U32).all()
