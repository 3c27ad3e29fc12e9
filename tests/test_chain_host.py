"""Which handles run all layers in one launch, and what happens below the workspace that takes (no GPU work)."""
import ctypes

import pytest

from paper_2211_13878_amd import binding


@pytest.fixture(scope="module")
def lib():
    return binding.load_library()


def create(lib, desc, n_bytes):
    h = ctypes.c_void_p(None)
    rc = lib.galv_dp_create(ctypes.byref(desc), ctypes.c_void_p(4096), n_bytes, ctypes.byref(h))
    if rc != binding.GALV_OK:
        return rc, None
    config = binding.galv_dp_get_config(h)
    lib.galv_dp_destroy(h)
    return rc, config


@pytest.mark.parametrize("B,L,S,E,chains", [(1, 37, 29, 9973, True), (8, 32, 22, 16384, True), (16, 48, 44, 2048, True), (1, 4, 6, 256, True),
                                            (32, 48, 22, 24576, False), (64, 96, 44, 32768, False), (8, 32, 65, 1000, False),
                                            (1, 1, 22, 5000, False), (40, 100, 44, 4000, True), (40, 20, 44, 4000, False), (12, 48, 44, 16384, False), (12, 24, 22, 16384, True)])
def test_the_rule_and_the_workspace(lib, B, L, S, E, chains):
    desc = binding.make_desc(B, L, S, E, 2, binding.GALV_DP_STREAMS(1))     # (no streams to create here)
    need, best = binding.galv_dp_workspace_bytes(desc), binding.galv_dp_workspace_bytes_preferred(desc)
    assert best >= need
    rc, config = create(lib, desc, best)
    assert rc == binding.GALV_OK and (config[0] == 2) == chains
    if L > 4:                                     # (with fewer layers all their rows may take less than a launch per layer)
        assert (best > need) == chains
    # less than preferred: a launch per layer; less than needed: refused
    for n_bytes in (best, best - 1, need):
        if n_bytes >= need:
            assert create(lib, desc, n_bytes)[0] == binding.GALV_OK
    if chains and L > 4:
        assert create(lib, desc, best - 1)[1][0] != 2
    assert create(lib, desc, 4096) == (binding.GALV_ERR_WORKSPACE, None)
    # what asks for a particular sweep, or for several streams, gets a launch per layer
    for flags in (binding.GALV_DP_FORCE_PACK, binding.GALV_DP_NO_PACK, binding.GALV_DP_BP_U8, binding.GALV_DP_NO_WIDE_TILES,
                  binding.GALV_DP_FORCE_WIDE_TILES, binding.GALV_DP_FORCE_PEEK, binding.GALV_DP_NO_PEEK, binding.GALV_DP_NO_U32,
                  binding.GALV_DP_STREAMS(2)):
        asked = binding.make_desc(B, L, S, E, 2, flags)
        assert binding.galv_dp_workspace_bytes_preferred(asked) == binding.galv_dp_workspace_bytes(asked)
        if flags != binding.GALV_DP_STREAMS(2):   # (streams are created with the handle, on a GPU)
            asked = binding.make_desc(B, L, S, E, 2, flags | binding.GALV_DP_STREAMS(1))
            rc, config = create(lib, asked, max(best, binding.galv_dp_workspace_bytes(asked)))
            assert rc == binding.GALV_OK and config[0] != 2
    # 64-bit integers asked for are an arithmetic, not a sweep
    asked = binding.make_desc(B, L, S, E, 2, binding.GALV_DP_FORCE_INT64 | binding.GALV_DP_STREAMS(1))
    rc, config = create(lib, asked, best)
    assert rc == binding.GALV_OK and (config[0] == 2) == chains


@pytest.mark.parametrize("B,L,S,E,peeks", [(1, 37, 29, 9973, 0), (3, 6, 22, 1500, 0), (1, 16, 64, 16000, 0), (16, 32, 12, 32768, 0),      # thin shapes; 16 strategies at most
                                           (8, 32, 22, 16384, 1), (11, 40, 30, 16384, 1), (8, 40, 44, 16384, 1), (11, 40, 60, 8192, 1)])
def test_the_configuration_says_whether_it_peeks(lib, B, L, S, E, peeks):
    """The fat shapes from 17 strategies on look at two cells of a row before they read it."""
    desc = binding.make_desc(B, L, S, E, 2, binding.GALV_DP_STREAMS(1))
    assert create(lib, desc, binding.galv_dp_workspace_bytes_preferred(desc))[1] == (2, peeks, 1, 128)


def test_preferred_checks_its_arguments(lib):
    n = ctypes.c_size_t(0)
    assert lib.galv_dp_workspace_bytes_preferred(None, ctypes.byref(n)) == binding.GALV_ERR_INVALID_ARG
    assert lib.galv_dp_workspace_bytes_preferred(ctypes.byref(binding.make_desc(1, 4, 6, 256)), None) == binding.GALV_ERR_INVALID_ARG


@pytest.mark.parametrize("S,E", [(2, 0), (8, 300), (44, 90)])
def test_no_wait_is_longer_than_a_bounded_number_of_layers(lib, S, E):
    """A wait inside the launch is given up after a fixed number of polls and may span a whole search: very deep searches take
    a launch per layer."""
    for L, chains in ((1023, True), (1024, True), (1025, False), (4096, False), (200000, False)):
        desc = binding.make_desc(1, L, S, E, 1, binding.GALV_DP_STREAMS(1))
        best = binding.galv_dp_workspace_bytes_preferred(desc)
        assert create(lib, desc, best)[1][0] == 2 if chains else create(lib, desc, best)[1][0] != 2, L


@pytest.mark.parametrize("B,L,S,E,chains", [(465, 2, 1, 16384, False), (465, 16, 1, 16384, False), (76, 4, 1, 100000, False), (3750, 8, 1, 2000, False),
                                            (625, 4, 6, 2000, False), (234, 2, 16, 2000, False), (1, 4, 44, 100000, False), (1, 16, 44, 100000, False),
                                            (93, 8, 2, 2000, True), (31, 16, 6, 2000, True), (3, 64, 6, 100000, True), (5000, 32, 1, 300, True),
                                            (64, 6, 1, 6000, True), (64, 6, 2, 6000, False), (64, 6, 9, 6000, True),
                                            # shares of 2048 and more: the rows that a shape adds count (33 strategies take 48)
                                            (3, 23, 33, 57599, False), (2, 23, 33, 57599, True), (3, 38, 33, 57599, True), (2, 23, 48, 57599, True)])
def test_layers_pay_for_the_workgroups(lib, B, L, S, E, chains):
    """Every tile costs a workgroup's start, which few layers do not pay for; a very large share of the budget per layer."""
    desc = binding.make_desc(B, L, S, E, 2, binding.GALV_DP_STREAMS(1))
    assert (create(lib, desc, binding.galv_dp_workspace_bytes_preferred(desc))[1][0] == 2) == chains


def test_the_larger_workspace_is_taken_only_where_there_is_room(lib):
    large = binding.make_desc(40, 100, 44, 4000, 2)                 # 3.1 and 9.2 GB
    need, best = binding.galv_dp_workspace_bytes(large), binding.galv_dp_workspace_bytes_preferred(large)
    assert best > 2 * need
    for least, free, want in ((False, 100 << 30, best), (False, 8 * (best - need), best), (False, 8 * (best - need) - 1, need),
                              (False, 0, need), (True, 1 << 40, need)):
        assert binding.workspace_size(large, least, lambda: free) == want
    small = binding.make_desc(8, 32, 22, 16384, 2)                   # less than 1 GB more: nobody is asked
    best = binding.galv_dp_workspace_bytes_preferred(small)
    assert best > binding.galv_dp_workspace_bytes(small)
    assert binding.workspace_size(small, False, None) == best
    assert binding.workspace_size(small, True, None) == binding.galv_dp_workspace_bytes(small)
    same = binding.make_desc(64, 96, 44, 32768, 2)                  # a launch per layer either way
    assert binding.workspace_size(same, True, None) == binding.workspace_size(same, False, None) == binding.galv_dp_workspace_bytes(same)
