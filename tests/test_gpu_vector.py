"""The fused s-exchange of equal blocks at the edges of its dispatch: the kernels for up to three and up to
five dimensions and the general one, one block per wavefront or not, tables in LDS or not, streaming loads,
both layouts.  The oracle says which rank each received block comes from (its exchange of rank numbers); the
blocks themselves are compared on the GPU, every byte."""
import numpy as np
import pytest
import torch

import iso_inputs as gen
import paper_1606_07676_amd as iso
from launch_paths import start_both_ways
from oracle import iso_oracle as orc

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _source_ranks(dims, offsets):
    """[p][s]: the rank whose block the oracle delivers as block i of rank R."""
    p, s = int(np.prod(dims)), len(offsets)
    ids = np.arange(p, dtype=np.int32).reshape(p, 1).view(np.uint8).copy()
    return orc.allgather(dims, offsets, ids).reshape(p, s, 4).view(np.int32)[:, :, 0]


def check_exchange(dims, offsets, op, alg, m, layout, send_off=0, recv_off=0):
    """One collective with the surroundings of receive buffer and workspace watched; returns nothing, raises on a wrong byte."""
    p, s = int(np.prod(dims)), len(offsets)
    a2a, slot = op == iso.ISO_OP_ALLTOALL, layout == iso.ISO_LAYOUT_SLOT_MAJOR
    comm = iso.iso_neighborhood_create(dims, np.asarray(offsets, np.int32).reshape(s, len(dims)))
    n_send, n_recv = p * m * (s if a2a else 1), p * s * m
    g = torch.Generator(device=DEV)
    g.manual_seed(p * 31 + s * 7 + m)
    send = torch.randint(0, 256, (n_send + send_off,), dtype=torch.uint8, device=DEV, generator=g)[send_off:]
    store = torch.full((n_recv + recv_off + 64,), 0xEE, dtype=torch.uint8, device=DEV)
    recv = store[recv_off:recv_off + n_recv]
    n_work = max(1, iso.iso_workspace_bytes(comm, op, alg, m))
    work_store = torch.full((n_work + 512,), 0xCC, dtype=torch.uint8, device=DEV)
    work = work_store[256:256 + n_work]
    init = iso.iso_neighbor_alltoall_init_layout if a2a else iso.iso_neighbor_allgather_init_layout
    req = init(send, recv, m, layout, work, comm, alg)
    start_both_ways(req, recv, work, starts=2)
    iso.iso_request_free(req)
    src = torch.from_numpy(_source_ranks(dims, offsets).astype(np.int64)).to(DEV)
    for i in range(s):
        got = recv.view(s, p, m)[i] if slot else recv.view(p, s, m)[:, i]
        if a2a:
            block = send.view(s, p, m)[i] if slot else send.view(p, s, m)[:, i]
        else:
            block = send.view(p, m)
        assert torch.equal(got, block.index_select(0, src[:, i])), (dims, m, layout, i)
    assert bool((store[:recv_off] == 0xEE).all()) and bool((store[recv_off + n_recv:] == 0xEE).all())
    assert bool((work_store[:256] == 0xCC).all()) and bool((work_store[256 + n_work:] == 0xCC).all()), (dims, m, layout)


TORI = [((700,), [(1,), (-3,), (0,), (699,)]), ((37, 21), gen.moore(2, 1)), ((1, 60), [(1, 1), (0, -2)]),
        ((7, 5, 11), gen.moore(3, 1)), ((3, 5, 4, 6), gen.von_neumann(4, 1)),
        ((3, 4, 2, 5, 3), gen.random_distinct(5, -3, 3, 20, 5)), ((2, 3, 2, 3, 2, 4), gen.von_neumann(6, 1)),
        ((6, 5, 5), gen.random_distinct(3, -3, 3, 129, 8))]           # one entry more than the LDS table takes


@pytest.mark.parametrize("layout", [iso.ISO_LAYOUT_RANK_MAJOR, iso.ISO_LAYOUT_SLOT_MAJOR])
@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("torus", range(len(TORI)))
def test_fused_exchange_over_dimensions_and_block_sizes(torus, op, layout):
    dims, offsets = TORI[torus]
    for m in (3, 16, 100, 1024, 1040, 3072):
        check_exchange(dims, offsets, op, iso.ISO_ALG_SX_FUSED, m, layout, recv_off=16)
    check_exchange(dims, offsets, op, iso.ISO_ALG_SX_FUSED, 2048, layout, send_off=5, recv_off=3)


@pytest.mark.parametrize("m", [8192, 8200])
def test_send_buffers_beyond_the_last_level_cache(m):
    """More than 256 MiB to send: streaming loads, in both forms of the kernel."""
    check_exchange((64, 65), gen.moore(2, 1), iso.ISO_OP_ALLTOALL, iso.ISO_ALG_SX_FUSED, m, iso.ISO_LAYOUT_RANK_MAJOR)


@pytest.mark.parametrize("dims,s,m,layout", [
    ((8, 9, 8, 7, 5), 9, 1024, iso.ISO_LAYOUT_RANK_MAJOR),       # far neighbours, whole lines: push, 20.6 MB to send
    ((8, 9, 8, 7, 5), 9, 1040, iso.ISO_LAYOUT_RANK_MAJOR),       # no whole lines: pull
    ((61, 64, 33), 7, 128, iso.ISO_LAYOUT_RANK_MAJOR),
    ((33, 31, 35), 6, 896, iso.ISO_LAYOUT_SLOT_MAJOR),           # 32 MB to send: push, groups of 4 entries and of 2
    ((33, 31, 35), 1, 997, iso.ISO_LAYOUT_SLOT_MAJOR),
    ((300, 301), 8, 331, iso.ISO_LAYOUT_SLOT_MAJOR),
    ((5, 6, 4, 7, 41), 5, 1024, iso.ISO_LAYOUT_SLOT_MAJOR)])
def test_allgather_forms_follow_where_the_reads_are_found(dims, s, m, layout):
    offsets = gen.random_distinct(len(dims), -3, 3, s, 17)
    check_exchange(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_SX_FUSED, m, layout, recv_off=128)


@pytest.mark.parametrize("alg", [iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM, iso.ISO_ALG_COMBINED_STAGED])
@pytest.mark.parametrize("dims,offsets,m,layout", [
    ((41, 40, 39), gen.moore(3, 1), 64, iso.ISO_LAYOUT_RANK_MAJOR),          # whole sectors: one read for two children
    ((41, 40, 39), gen.moore(3, 1), 80, iso.ISO_LAYOUT_RANK_MAJOR),          # not: every child reads for itself
    ((53, 67), gen.moore(2, 2) + [(0, 0), (1, 2), (1, 2)], 1056, iso.ISO_LAYOUT_RANK_MAJOR),   # repeated neighbours
    ((29, 31, 17), gen.moore(3, 1) + [(2, 0, 0), (2, 1, 0), (-2, 0, 1)], 100, iso.ISO_LAYOUT_SLOT_MAJOR),
    ((300, 299), gen.von_neumann(2, 2), 5, iso.ISO_LAYOUT_SLOT_MAJOR),
    ((2, 3, 1, 29, 211), gen.von_neumann(5, 1), 192, iso.ISO_LAYOUT_RANK_MAJOR)])   # sides of 1, 2 and 3: both ways alias
def test_allgather_rounds_that_read_a_block_once_for_all_its_children(dims, offsets, m, layout, alg):
    check_exchange(dims, [tuple(c) for c in offsets], iso.ISO_OP_ALLGATHER, alg, m, layout, recv_off=64)


@pytest.mark.parametrize("alg", [iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_STAGED])
@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("dims,offsets,m,layout", [
    ((24, 25, 23), gen.moore(3, 1), 450, iso.ISO_LAYOUT_RANK_MAJOR),     # 161 MB: between half the last-level cache and all
    ((24, 25, 23), gen.moore(3, 1), 450, iso.ISO_LAYOUT_SLOT_MAJOR),
    ((24, 25, 23), gen.moore(3, 1), 1001, iso.ISO_LAYOUT_RANK_MAJOR),    # 359 MB: beyond it
    ((24, 25, 23), gen.moore(3, 1), 1024, iso.ISO_LAYOUT_SLOT_MAJOR),
    ((61, 70), gen.moore(2, 2), 3000, iso.ISO_LAYOUT_RANK_MAJOR),        # ranks in groups
    ((7, 6, 41), gen.random_distinct(3, -3, 3, 140, 2), 1300, iso.ISO_LAYOUT_RANK_MAJOR)])   # tables beyond LDS
def test_rounds_by_what_the_last_level_cache_holds(dims, offsets, m, layout, op, alg):
    check_exchange(dims, [tuple(c) for c in offsets], op, alg, m, layout, recv_off=3)


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("m", [400, 1000])
def test_mesh_rounds_by_what_the_last_level_cache_holds(m, op):
    dims, periodic, offsets = (25, 24, 26), (False, True, False), gen.moore(3, 1)
    p, s, a2a = int(np.prod(dims)), len(offsets), op == iso.ISO_OP_ALLTOALL
    comm = iso.iso_neighborhood_create_mesh(dims, periodic, np.asarray(offsets, np.int32))
    send = torch.randint(0, 256, (p, s if a2a else 1, m), dtype=torch.uint8, device=DEV)
    recv = torch.full((p, s, m), 0xEE, dtype=torch.uint8, device=DEV)
    work = torch.empty(max(1, iso.iso_workspace_bytes(comm, op, iso.ISO_ALG_COMBINED, m)), dtype=torch.uint8, device=DEV)
    init = iso.iso_neighbor_alltoall_init if a2a else iso.iso_neighbor_allgather_init
    req = init(send, recv, m, work, comm, iso.ISO_ALG_COMBINED)
    iso.iso_start(req)
    iso.iso_wait(req)
    iso.iso_request_free(req)
    src, valid = orc.source_ranks_mesh(dims, periodic, offsets)
    for i in range(s):
        v = torch.from_numpy(np.ascontiguousarray(valid[:, i])).to(DEV)
        at = torch.from_numpy(np.where(valid[:, i], src[:, i], 0).astype(np.int64)).to(DEV)
        want = send[:, i if a2a else 0].index_select(0, at)
        want[~v] = 0xEE
        assert torch.equal(recv[:, i], want), (m, i)


CHAINS = [((8, 8), gen.moore(2, 1), (1, 7, 32, 64, 1000, 8192, 8200)), ((8, 8, 8), gen.moore(3, 1), (2, 16, 40, 64, 144)),
          ((2048,), [(1,), (-5,), (0,), (2047,)], (16, 20, 36, 64)), ((64, 64), [(0, 1), (-1, 0), (0, 0)], (16, 33, 48)),
          ((45, 91), [(1, 1), (3, -2)], (16, 17, 8)), ((3, 1, 2, 5, 2, 3, 2, 2), gen.von_neumann(8, 1), (12, 100, 112)),
          ((4, 3), [(1, 1), (1, 1), (0, 0), (0, 0), (5, -7), (2, 0)], (5, 16, 100000)),
          ((17, 19), gen.random_distinct(2, -3, 3, 36, 6), (64, 100, 208)),       # 72 hops and fewer
          ((7, 3, 15, 7), gen.random_distinct(4, -2, 2, 1, 3), (4100,)),          # a column of one unit: not where it overlaps
          ((8, 8), [(1, 1), (0, 1), (2, 0)], (1040, 2000, 2056)),                 # two and three columns of 64 units, with and without an overlap
          ((4, 3), [(1, 1), (1, 1), (0, 0), (0, 0), (5, -7), (2, 0)], (5456, 5464, 10000)),
          ((5, 5, 5, 5), gen.von_neumann(4, 1), (100, 400, 1000)), ((16, 16), gen.von_neumann(2, 1), (2000, 3000))]


@pytest.mark.parametrize("alg", [iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM, iso.ISO_ALG_COMBINED_STAGED])
@pytest.mark.parametrize("layout", [iso.ISO_LAYOUT_RANK_MAJOR, iso.ISO_LAYOUT_SLOT_MAJOR])
@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("case", range(len(CHAINS)))
def test_small_collective_in_one_launch(case, op, layout, alg):
    dims, offsets, sizes = CHAINS[case]
    for m in sizes:
        check_exchange(dims, [tuple(c) for c in offsets], op, alg, m, layout, send_off=1, recv_off=5)


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("dims,m", [((23, 24, 25), 48), ((51, 52, 49), 48), ((51, 52, 49), 80), ((61, 62, 63), 80)])
def test_staged_schedule_by_what_the_last_level_cache_holds(dims, m, op):
    """17, 162, 270 and 496 MB of blocks."""
    check_exchange(dims, gen.moore(3, 1), op, iso.ISO_ALG_COMBINED_STAGED, m, iso.ISO_LAYOUT_RANK_MAJOR, recv_off=16)


@pytest.mark.parametrize("dims,edge,align", [((32, 32, 32), 25, 16), ((21, 20, 19), 51, 1), ((64, 63, 65), 12, 1), ((16, 17, 16, 17), 6, 4),
                                             ((31, 32, 33), (8, 200, 300, 400, 500), 1), ((31, 32, 33), (16, 144, 256, 400, 1024), 16)])
def test_small_and_large_blocks_by_their_size(dims, edge, align):
    """Blocks of up to 128 bytes and larger ones together, 64 MiB and more, against the straightforward exchange: sizes with a
    launch each, and too many of them for that, which the rounds' kernel takes by size."""
    offsets = gen.moore(len(dims), 1)
    p, sizes = int(np.prod(dims)), list(gen.stencil_block_sizes(offsets, edge) if isinstance(edge, int) else [edge[i % 5] for i in range(26)])
    displs, row = gen.packed_displacements(sizes, align)
    assert p * sum(sizes) > 64 << 20
    comm = iso.iso_neighborhood_create(dims, offsets)
    send = torch.randint(0, 256, (p * row,), dtype=torch.uint8, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(8))
    got = []
    for alg in (iso.ISO_ALG_SX_FUSED, iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        recv = torch.full((p * row,), 0xEE, dtype=torch.uint8, device="cuda:0")
        work = torch.empty(max(1, iso.iso_workspace_bytes_v(comm, iso.ISO_OP_ALLTOALL, alg, sizes)), dtype=torch.uint8, device="cuda:0")
        req = iso.iso_neighbor_alltoallv_init(send, sizes, displs, row, recv, sizes, displs, row, work, comm, alg)
        for _ in range(2):
            iso.iso_start(req)
        iso.iso_wait(req)
        iso.iso_request_free(req)
        got.append(recv)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
