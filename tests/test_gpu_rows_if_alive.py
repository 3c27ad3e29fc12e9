"""Instances on 64-bit keys of a handle that keeps the byte table by default: those whose transition costs
dwarf the spread of the layer costs keep cost rows instead, the others do not, in one batch and from one solve
of a handle to the next.  Compared with the oracle, whole tables for some instances."""
import numpy as np
import pytest

import oracle
from paper_2211_13878_amd import binding, workloads
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


def workload(S, B, L, E, seed, dear, c_hi=1 << 32):
    w = workloads.random_workload(seed, B, L, S, E, nR=2, m_range=(0, 2 * E // L), c_range=(0, c_hi), r_range=(0, c_hi // 40),
                                  infeasible=0.05, zero_diagonal=False)
    w.R[dear] *= 38                                # just below 2^32: nearly every row stays alive
    w.budget[:] = np.linspace(E - 130, E, B).astype(np.int32)
    return w


@pytest.mark.parametrize("S,B,L,E", [(14, 8, 5, 13000), (22, 8, 6, 8100), (44, 6, 5, 5500), (64, 6, 5, 4100), (130, 16, 4, 2100)])
@pytest.mark.parametrize("c_hi,status", [(1 << 32, binding.GALV_INSTANCE_OK_FAST_WIDE), (1 << 27, binding.GALV_INSTANCE_OK_FAST)])
def test_both_kinds_in_one_batch_and_in_turn(S, B, L, E, c_hi, status):
    flags = binding.GALV_DP_NO_U32
    dear = [b for b in range(B) if b % 3 != 1]
    w = workload(S, B, L, E, 5 * S, dear, c_hi)
    sol = binding.Solver(B, L, S, E, w.nR, flags)
    assert sol.config()["packed"] == 1             # (the handle's choice; the instances' is the preparation's)
    sol.close()
    check_against_oracle(w, flags=flags, table_instances=[0, 1], threads=8, expect_status=status)
    sol = binding.Solver(B, L, S, E, w.nR, flags)
    for seed, kind in ((1, []), (2, list(range(B))), (3, dear), (4, [b for b in range(B) if b not in dear])):
        w = workload(S, B, L, E, 7 * S + seed, kind, c_hi)
        cost, last = sol.solve(*binding.upload(w))
        plan = sol.backtrack().cpu().numpy()
        best, _ = sol.best_per_budget()
        for b, ref in enumerate(oracle.solve_workload(w, threads=8)):
            assert int(cost[b]) == ref.best_cost and int(last[b]) == ref.best_last and (plan[b] == ref.plan).all()
            assert int(best[b, int(w.budget[b])]) == ref.best_cost
    sol.close()
