"""The sweep shapes by launch size: tiles split over more waves (few tiles), the plain shape
(GALV_DP_NO_WIDE_TILES asks for it) and the finest split (very few tiles of 17 to 32 strategies), at the
edges of the strategy counts that each covers, over cost rows and byte tables, with 32-bit keys, 8-byte
cells and 64-bit keys in one batch.  Whole tables are compared with the oracle's."""
import pytest

from paper_2211_13878_amd import binding, workloads
from test_gpu_parity import check_against_oracle, oracle_refs

pytestmark = pytest.mark.gpu
PACK, PEEK, NO_PEEK, ROWS, NORMAL = (binding.GALV_DP_FORCE_PACK, binding.GALV_DP_FORCE_PEEK, binding.GALV_DP_NO_PEEK,
                                     binding.GALV_DP_NO_PACK, binding.GALV_DP_NO_WIDE_TILES)


@pytest.mark.parametrize("S", [1, 8, 9, 16, 17, 24, 25, 32, 33, 48, 49, 64, 65, 128, 129])
@pytest.mark.parametrize("B", [3, 66])                       # (12 and 264 tiles: the finest split takes up to 256)
def test_shapes_by_launch_size(S, B):
    w = workloads.random_workload(31 * S + B, B, 4, S, 500, nR=2, m_range=(0, 150), c_range=(0, 3000), r_range=(0, 400),
                                  infeasible=0.08, zero_diagonal=False)
    w.c[1] <<= 30                                            # 8-byte cells
    w.R[2] <<= 20                                            # 64-bit keys
    w.budget[:3] = (500, 383, 384)
    tables = [0, 1, 2]
    refs = oracle_refs(w, list(range(B)), tables, (), 8)
    for flags in (PACK | PEEK, PACK | NO_PEEK, ROWS | PEEK, ROWS | NO_PEEK, PACK | PEEK | NORMAL, ROWS | NO_PEEK | NORMAL):
        check_against_oracle(w, flags=flags, table_instances=tables, refs=refs, allow_vacuous=S == 1)


def test_a_shape_at_the_limit_of_the_fixed_workspace_is_still_taken():
    """The split shapes pad 22 strategies to 24: where only the plain shape fits the fixed workspace, it is kept."""
    E = max(e for e in range(1023, 60000, 1024)
            if binding.galv_dp_workspace_bytes(binding.make_desc(1, 4, 22, e, 1, NORMAL)) <= binding.GALV_DP_STATIC_BYTES)
    assert binding.galv_dp_workspace_bytes(binding.make_desc(1, 4, 22, E)) <= binding.GALV_DP_STATIC_BYTES
    assert binding.galv_dp_workspace_bytes(binding.make_desc(1, 4, 22, E + 1024)) > binding.GALV_DP_STATIC_BYTES
