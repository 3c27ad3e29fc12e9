"""The sweep that takes all layers of a small search in one launch: workgroups own budget columns and pass a layer's
cells on to their neighbours.  Edges of the strategy counts that each shape covers, of tiles and of budgets, every
arithmetic path in one batch, more workgroups than the GPU holds at a time, and solves that overlap on several streams.
Whole tables are compared with the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_13878_amd import binding, workloads
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


def workload(seed, B, L, S, E, m_hi=None, nR=2):
    return workloads.random_workload(seed, B, L, S, E, nR=nR, m_range=(0, m_hi or 2 * E // L), c_range=(0, 3000), r_range=(0, 400),
                                     infeasible=0.08, zero_diagonal=False)


def mixed(w):
    """Instances of every status: 32-bit keys, 8-byte cells, 64-bit keys over 32-bit and over larger costs, 64-bit
    integers, one with an invalid value, and 64-bit keys with transition costs beyond 32 bits."""
    w.c[1] <<= 30
    w.R[2] <<= 20
    w.c[3] <<= 30
    w.R[3] <<= 20
    w.c[4] <<= 46
    w.R[4] <<= 34
    w.R[5, 0, 0, 0] = -1
    w.c[6] <<= 30
    w.R[6] <<= 25
    return w


@pytest.mark.parametrize("S", [1, 2, 8, 9, 16, 17, 24, 25, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("B,E", [(7, 700), (150, 640)])      # thin waves, and from 353, 705 or 769 tiles on fat ones
def test_strategy_counts_and_arithmetic_paths(S, B, E):
    w = mixed(workload(17 * S + B, B, 5, S, E))
    w.budget[:7] = (E, 383, 384, E, E, E, E)
    some = list(range(7)) + list(range(7, B, 29))
    bad = 5
    cost, last, plan, status = check_against_oracle(w, table_instances=[0, 1, 2, 3, 4, 6], oracle_instances=[b for b in some if b != bad],
                                                    threads=8, allow_vacuous=S == 1)
    assert status[bad] == binding.GALV_INSTANCE_BAD_VALUE and cost[bad] == binding.GALV_INF and (plan[bad] == -1).all()
    if S >= 8:
        assert set(status[:5]) == {0, 1, 2, 3, 4}


@pytest.mark.parametrize("E", [0, 1, 126, 127, 128, 129, 255, 256, 1023, 4099])
@pytest.mark.parametrize("L", [2, 3, 9])
def test_edges_of_tiles_and_budgets(L, E):
    w = workload(1000 + 31 * L + E, 5, L, 22, E, m_hi=max(1, E // L))
    w.budget[:] = (E, max(0, E - 1), E // 2, min(E, 128), 0)
    w.c[1] <<= 30
    w.r_idx[:, 1:] = np.arange(L - 1) % 2                    # the transition matrix changes from layer to layer
    check_against_oracle(w, table_instances=list(range(5)), threads=8, allow_vacuous=True)


@pytest.mark.parametrize("m_hi", [3, 40, 900, 6000])
def test_memories_from_within_a_tile_to_most_of_the_budget(m_hi):
    w = workload(77 + m_hi, 3, 12, 29, 5003, m_hi=m_hi)
    w.m[1, 3, :] = 5004                                      # a layer without a usable strategy
    check_against_oracle(w, table_instances=[0, 1, 2], threads=8)


def test_nothing_can_be_left_out():
    """Every row stays alive in every tile, with each kind of key."""
    for S in (16, 24, 48, 64):
        w = workloads.random_workload(300 + S, 3, 6, S, 900, nR=2, m_range=(0, 150), c_range=(0, 9), r_range=(1000, 5000),
                                      infeasible=0.05, zero_diagonal=False)
        w.c[1] <<= 36
        w.R[1] <<= 18
        check_against_oracle(w, table_instances=[0, 1], threads=8)


@pytest.mark.parametrize("B,L,S,E", [(300, 6, 6, 3000), (1, 4, 22, 150000), (90, 7, 44, 1100),
                                     (300, 27, 6, 3000), (1, 70, 2, 280000), (90, 17, 44, 1100)])      # these in one launch
def test_more_workgroups_than_the_gpu_holds(B, L, S, E):
    w = workload(5 * B + S, B, L, S, E)
    w.c[::3] <<= 30
    desc = binding.make_desc(B, L, S, E, 2)
    assert L < 10 or binding.galv_dp_workspace_bytes_preferred(desc) > binding.galv_dp_workspace_bytes(desc)
    check_against_oracle(w, oracle_instances=list(range(0, B, 37)), table_instances=[0] if L < 30 else [], threads=8)


def test_solves_that_overlap_on_several_streams():
    """Three handles on three streams at once, with changing inputs: each solve waits for its own words only."""
    shapes = [(2, 9, 22, 9000), (6, 14, 12, 3000), (1, 6, 48, 12000)]
    jobs = []
    for i, (B, L, S, E) in enumerate(shapes):
        ws = [workload(900 + 10 * i + j, B, L, S, E) for j in range(3)]
        jobs.append((binding.Solver(B, L, S, E, 2), [binding.upload(w) for w in ws],
                     [oracle.solve_workload(w, threads=8) for w in ws], torch.cuda.Stream(), []))
    torch.cuda.synchronize()
    for rep in range(12):
        for sol, devs, refs, stream, got in jobs:
            with torch.cuda.stream(stream):
                cost, _ = sol.solve(*devs[rep % 3])
                plan = sol.backtrack()
                got.append((cost.clone(), plan.clone()))
    torch.cuda.synchronize()
    for sol, devs, refs, stream, got in jobs:
        for rep, (cost, plan) in enumerate(got):
            for b, ref in enumerate(refs[rep % 3]):
                assert int(cost[b]) == ref.best_cost and (plan[b].cpu().numpy() == ref.plan).all(), (rep, b)
        sol.close()


def test_a_graph_that_is_replayed_with_changing_inputs():
    B, L, S, E = 4, 11, 22, 6000
    ws = [workload(700 + j, B, L, S, E) for j in range(3)]
    devs = [binding.upload(w) for w in ws]
    sol = binding.Solver(B, L, S, E, 2)
    inputs = [t.clone() for t in devs[0]]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        sol.solve(*inputs), sol.backtrack()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cost, _ = sol.solve(*inputs)
        plan = sol.backtrack()
    for rep in range(6):
        for to, t in zip(inputs, devs[rep % 3]):
            to.copy_(t)
        graph.replay()
        torch.cuda.synchronize()
        for b, ref in enumerate(oracle.solve_workload(ws[rep % 3], threads=4)):
            assert int(cost[b]) == ref.best_cost and (plan[b].cpu().numpy() == ref.plan).all(), (rep, b)
    sol.close()


def test_without_the_memory_for_all_layers_a_launch_per_layer(monkeypatch):
    w = workload(5, 2, 9, 22, 4000)
    desc = binding.make_desc(w.B, w.L, w.S, w.E_max, w.nR)
    best, need = binding.galv_dp_workspace_bytes_preferred(desc), binding.galv_dp_workspace_bytes(desc)
    assert best > need
    empty = torch.empty

    def scarce(*size, **options):
        if size == (best,):
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(*size, **options)

    results = []
    for chained in (True, False):
        if not chained:
            monkeypatch.setattr(binding.torch, "empty", scarce)
        sol = binding.Solver(w.B, w.L, w.S, w.E_max, w.nR)
        assert sol.workspace_bytes == (best if chained else need) and (sol.config()["packed"] == 2) == chained
        dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (w.c, w.m, w.R, w.r_idx, w.budget)]
        cost, last = sol.solve(*dev)
        results.append([x.cpu().numpy().copy() for x in (cost, last, sol.backtrack())])
        sol.close()
    for x, y in zip(*results):
        assert (x == y).all()


def test_the_least_workspace_on_request_and_where_little_is_left(monkeypatch):
    w = workload(6, 8, 60, 22, 20000)
    dev = binding.upload(w)
    results = []
    for least, left in ((False, None), (True, None), (False, 1 << 28)):
        if left:
            monkeypatch.setattr(binding, "_free_bytes", lambda device: left)
        sol = binding.Solver(w.B, w.L, w.S, w.E_max, w.nR, least_workspace=least)
        small = least or left is not None
        assert sol.workspace_bytes == sol.workspace.numel()
        assert (sol.workspace_bytes == binding.galv_dp_workspace_bytes(sol.desc)) == small and (sol.config()["packed"] == 2) == (not small)
        cost, last = sol.solve(*dev)
        results.append([x.cpu().numpy().copy() for x in (cost, last, sol.backtrack())])
        sol.close()
    for r in results[1:]:
        assert all((x == y).all() for x, y in zip(r, results[0]))


@pytest.mark.parametrize("S", [1, 7, 16, 22, 29, 44, 64])      # every row count that a wave covers, with and without a remainder
@pytest.mark.parametrize("m_hi", [0, 40, 900, 5003])           # from the own block only to blocks that nothing reaches
def test_whole_costs(S, m_hi):
    """Transition costs beyond a relative cost of 32 bits (keys in doubles), and costs beyond a key (64-bit integers)."""
    w = workload(4000 + 7 * S + m_hi, 4, 6, S, 1500, m_hi=max(1, m_hi))
    if m_hi == 0:
        w.m[:] = 0
    w.m[:, :, S // 2:] //= 40                                  # (some strategies fit whatever m_hi is: six layers, a budget of 1500)
    w.m[1, 2, :] = 1501                                        # a layer without a usable strategy
    w.m[2:, 1::2, 0] = 129                                     # a shift of one column more than a block
    w.budget[:] = (1500, 1500, 1407, 128)
    w.r_idx[:, 1:] = np.arange(5) % 2
    w.R[:2] = (w.R[:2] << 24) + (1 << 32)
    w.c[2:] <<= 44
    w.R[2:] <<= 40
    _, _, _, status = check_against_oracle(w, table_instances=[0, 1, 2, 3], threads=8, allow_vacuous=S == 1)
    assert list(status) == [binding.GALV_INSTANCE_OK_FAST_WIDE] * 2 + [binding.GALV_INSTANCE_OK_INT64] * 2


@pytest.mark.parametrize("S", [3, 22, 44, 64])
def test_the_largest_transition_costs_and_keys(S):
    """The largest relative cost that 32 bits hold and one more; the largest plan cost that a key holds and one more; a matrix
    that no layer uses with entries above every plan cost."""
    k = max(1, (S - 1).bit_length())
    w = workload(600 + S, 5, 3, S, 700)
    w.r_idx[:] = 0
    w.R[0, 0, 0, S - 1], w.R[1, 0, 0, S - 1] = (1 << 32) - 2, (1 << 32) - 1
    w.c[:2] <<= 32
    most = (1 << (52 - k)) - 1                    # bound of all plan costs: the layers' largest plus two transitions
    for b, top in ((2, most), (3, most + 1)):
        layers = int(w.c[b].max(axis=1).sum())
        w.c[b, 0, np.argmax(w.c[b, 0])] += (top - layers) % 2
        w.R[b, 0, S - 1, 0] = w.R[b, 0, 0, 0] = w.R[b, 0, 0, S - 1] = (top - layers) // 2
    w.R[4, 1] = 1 << 55
    _, _, _, status = check_against_oracle(w, table_instances=[0, 1, 2, 3, 4], threads=8)
    wide, integers = binding.GALV_INSTANCE_OK_FAST_WIDE, binding.GALV_INSTANCE_OK_INT64
    assert list(status) == [wide, wide, wide, integers, wide]


@pytest.mark.parametrize("S", [1, 8, 12, 16, 22, 29, 32, 44, 48, 60, 64])
@pytest.mark.parametrize("B,E", [(3, 900), (110, 900)])        # thin and fat shapes
def test_matrices_that_change_at_every_layer(S, B, E):
    w = workload(800 + S + B, B, 8, S, E, nR=3)
    w.r_idx[:, 1:] = np.arange(1, 8) % 3
    w.r_idx[2, 1:] = (0, 0, 2, 1, 1, 2, 2)
    w.c[1] <<= 30
    w.R[2] <<= 20
    check_against_oracle(w, table_instances=[0, 1, 2], oracle_instances=[0, 1, 2, B - 1], threads=8, allow_vacuous=S == 1)


@pytest.mark.parametrize("S,nR,L", [(8, 33, 70), (29, 9, 30), (64, 5, 16)])      # slots for 32 or 16, 8 or 4, 4 or 2 matrices
def test_more_matrices_than_the_unlimited_recurrence_keeps(S, nR, L):
    """Matrices come back after another one has taken their slot, next to ones that stay."""
    w = workload(900 + S, 3, L, S, 1200, nR=nR)
    w.r_idx[:, 1:] = (np.arange(L - 1) * 3 + np.arange(L - 1) // 7) % nR
    w.r_idx[1, 1:] = np.where(np.arange(L - 1) % 2, 0, nR - 1)           # two that share a slot, in turns
    w.R[2] <<= 20
    check_against_oracle(w, table_instances=[0, 1, 2], threads=8)
