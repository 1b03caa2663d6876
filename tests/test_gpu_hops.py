"""Collectives whose blocks go through all their hops in one launch, every stop stored: the kernels for up to three and up to
five dimensions, one block per wavefront or not, last units that overlap, both layouts and orders, against the oracle, and
against the launches of the rounds."""
import numpy as np
import pytest
import torch

import iso_inputs as gen
import paper_1606_07676_amd as iso
from launch_paths import start_both_ways
from oracle import iso_oracle as orc
from test_gpu_vector import check_exchange

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RANK, SLOT = iso.ISO_LAYOUT_RANK_MAJOR, iso.ISO_LAYOUT_SLOT_MAJOR
COMBINED, BYDIM = iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM


@pytest.mark.parametrize("dims,offsets,m,layout,alg,send_off,recv_off", [
    ((23, 24, 25), gen.moore(3, 1), 128, RANK, COMBINED, 0, 0),
    ((23, 24, 25), gen.moore(3, 1), 128, RANK, COMBINED, 5, 3),
    ((19, 20, 21), gen.moore(3, 1), 1027, RANK, COMBINED, 0, 7),
    ((31, 29, 30), gen.von_neumann(3, 2), 321, RANK, COMBINED, 0, 0),
    ((61, 67), gen.von_neumann(2, 2) + [(0, 0), (1, 2), (1, 2)], 1024, RANK, COMBINED, 0, 0),       # repeated and zero
    ((11, 12, 13, 9), gen.random_distinct(4, -3, 3, 30, 5), 640, RANK, COMBINED, 0, 0),
    ((7, 6, 5, 8, 9), gen.random_distinct(5, -3, 3, 40, 5), 2048, RANK, COMBINED, 0, 1),            # block by block
    ((7, 6, 5, 8, 9), gen.random_distinct(5, -3, 3, 40, 5), 128, RANK, COMBINED, 0, 0),
    ((2, 3, 1, 29, 211), gen.random_distinct(5, -3, 3, 40, 6), 520, RANK, COMBINED, 0, 0),          # sides of 1, 2 and 3 alias
    ((6, 5, 5, 7), gen.random_distinct(4, -3, 3, 128, 8), 384, RANK, COMBINED, 0, 0),               # a full table
    ((6, 5, 5, 7), gen.random_distinct(4, -3, 3, 129, 8), 384, RANK, COMBINED, 0, 0),               # one more: its rounds
    ((23, 24, 25), gen.moore(3, 1), 256, SLOT, COMBINED, 1, 0),
    ((29, 31, 27), gen.moore(3, 1), 107, SLOT, COMBINED, 0, 2),
    ((8, 7, 9, 6, 5), gen.random_distinct(5, -3, 3, 40, 5), 1024, SLOT, COMBINED, 0, 0),
    ((9, 10, 11), gen.moore(3, 1), 256, RANK, BYDIM, 0, 0),
    ((41, 40, 39), gen.moore(3, 1), 320, RANK, BYDIM, 0, 0)])
def test_alltoall_through_all_hops(dims, offsets, m, layout, alg, send_off, recv_off):
    check_exchange(dims, [tuple(int(x) for x in c) for c in offsets], iso.ISO_OP_ALLTOALL, alg, m, layout, send_off, recv_off)


@pytest.mark.parametrize("dims,offsets,m,layout,alg,send_off,recv_off", [
    ((23, 24, 25), gen.moore(3, 1), 128, RANK, COMBINED, 0, 0),                                      # all nodes are receive blocks
    ((23, 24, 25), gen.moore(3, 1), 257, RANK, COMBINED, 3, 1),
    ((61, 67), gen.moore(2, 2) + [(0, 0), (1, 2), (1, 2)], 1024, RANK, COMBINED, 0, 0),
    ((23, 24, 25), gen.random_distinct(3, -3, 3, 20, 5) + [(0, 0, 0), (2, -2, 1), (2, -2, 1)], 1000, RANK, COMBINED, 0, 0),
    ((7, 6, 5, 8, 9), gen.random_distinct(5, -3, 3, 40, 5), 128, RANK, COMBINED, 0, 0),              # pull, an order of its own
    ((8, 9, 8, 7, 5), gen.random_distinct(5, -3, 3, 36, 7), 1152, RANK, COMBINED, 0, 0),             # push
    ((8, 9, 8, 7, 5), gen.random_distinct(5, -3, 3, 36, 7), 1152, RANK, COMBINED, 0, 16),
    ((8, 9, 8, 7, 5), gen.random_distinct(5, -3, 3, 36, 7), 1025, RANK, COMBINED, 0, 16),
    ((2, 3, 1, 29, 211), gen.random_distinct(5, -3, 3, 30, 6), 640, RANK, COMBINED, 0, 0),
    ((9, 8, 7, 11), gen.random_distinct(4, -3, 3, 30, 5), 100, SLOT, COMBINED, 0, 0),                # push, 2 at a time
    ((33, 31, 35), gen.random_distinct(3, -3, 3, 9, 5), 900, SLOT, COMBINED, 0, 5),                  # 4 at a time
    ((23, 24, 25), gen.moore(3, 1), 16, SLOT, COMBINED, 0, 0),
    ((17, 18, 19), gen.moore(3, 1), 33, RANK, COMBINED, 0, 1),
    ((31, 32, 7), gen.random_distinct(3, -3, 3, 20, 5), 47, RANK, BYDIM, 0, 0),
    ((41, 40, 39), gen.moore(3, 1), 320, RANK, BYDIM, 0, 0),
    ((8, 9, 8, 7, 5), gen.random_distinct(5, -3, 3, 36, 7), 1024, RANK, BYDIM, 0, 0)])
def test_allgather_through_all_hops(dims, offsets, m, layout, alg, send_off, recv_off):
    check_exchange(dims, [tuple(int(x) for x in c) for c in offsets], iso.ISO_OP_ALLGATHER, alg, m, layout, send_off, recv_off)


@pytest.mark.parametrize("dims,n,m,send_off,recv_off", [((9, 8, 8, 9, 8), 40, 16, 0, 0), ((7, 8, 7, 6, 7), 40, 17, 1, 3), ((11, 12, 11, 13), 30, 63, 0, 0),
                                                        ((12, 12, 11, 12, 12), 10, 21, 5, 0)])
def test_small_allgather_blocks_and_many_nodes(dims, n, m, send_off, recv_off):
    """Plain stores, under a sector: whole units and last units that overlap, any address."""
    offsets = [tuple(int(x) for x in c) for c in gen.random_distinct(len(dims), -3, 3, n, 160607676)]
    check_exchange(dims, offsets, iso.ISO_OP_ALLGATHER, COMBINED, m, RANK, send_off, recv_off)


@pytest.mark.parametrize("dims,offsets,m,send_off,recv_off", [((20, 21, 24), gen.moore(3, 1), 901, 0, 5), ((29, 31, 27), gen.moore(3, 1)[:25], 272, 3, 0),
                                                              ((10, 11, 9, 8), gen.von_neumann(4, 2), 1040, 0, 0), ((181, 177), gen.moore(2, 1) + [(0, 0)], 210, 0, 0)])
def test_slot_major_allgathers_pushed_two_at_a_time(dims, offsets, m, send_off, recv_off):
    """All nodes are receive blocks, an even and an odd number of them."""
    check_exchange(dims, [tuple(int(x) for x in c) for c in offsets], iso.ISO_OP_ALLGATHER, COMBINED, m, SLOT, send_off, recv_off)


@pytest.mark.parametrize("m", [4224, 4480 + 16])
def test_two_dimensional_allgather_of_more_than_the_cache_holds(m):
    """Whole lines, pushed from a window that the L2 holds; parts of lines, a launch per dimension."""
    check_exchange((260, 257), [tuple(int(x) for x in c) for c in gen.moore(2, 1)], iso.ISO_OP_ALLGATHER, COMBINED, m, RANK)


@pytest.mark.parametrize("layout", [RANK, SLOT])
def test_equal_blocks_of_the_irregular_call_with_empty_ones(layout):
    """Every third block empty, rows with gaps: those bytes and blocks stay as they are."""
    dims, offsets, m = (23, 24, 25), gen.moore(3, 1), 640
    p, s = int(np.prod(dims)), len(offsets)
    sizes = [0 if i % 3 == 0 else m for i in range(s)]
    step = p * m + 48 if layout == SLOT else m + 48
    displs = [i * step for i in range(s)]
    extent, n = (0, s * step) if layout == SLOT else (s * step, p * s * step)
    send = torch.randint(0, 256, (n,), dtype=torch.uint8, device=DEV, generator=torch.Generator(DEV).manual_seed(2))
    comm, got = iso.iso_neighborhood_create(dims, offsets), []
    for alg in (iso.ISO_ALG_SX_FUSED, COMBINED):
        recv = torch.full((n,), 0xEE, dtype=torch.uint8, device=DEV)
        work = torch.empty(max(1, iso.iso_workspace_bytes_v(comm, iso.ISO_OP_ALLTOALL, alg, sizes)), dtype=torch.uint8, device=DEV)
        req = iso.iso_neighbor_alltoallv_init_layout(send, sizes, displs, extent, recv, sizes, displs, extent, layout, work, comm, alg)
        assert iso.iso_request_start_info(req)["kernels"] == 1
        iso.iso_start(req)
        iso.iso_wait(req)
        iso.iso_request_free(req)
        got.append(recv)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("dims,periodic,offsets,sizes", [
    ((25, 24, 26), (0, 1, 0), gen.moore(3, 1) + [(0, 0, 0), (25, 0, 1), (-30, 2, 0), (2, 25, -2)], (128, 333, 1024)),
    ((130, 71), (0, 0), gen.moore(2, 2) + [(129, -70)], (128, 520)),
    ((7, 6, 9, 5, 8), (1, 0, 0, 1, 0), gen.random_distinct(5, -3, 3, 40, 5), (256, 2048)),
    ((3, 2, 1, 60, 33), (0, 0, 0, 0, 1), gen.random_distinct(5, -3, 3, 30, 6), (640,))])
def test_boxes(dims, periodic, offsets, sizes, op):
    """Dimensions that do not wrap: the same launches for one launch per dimension, and the straightforward exchange with the
    tables of a torus; receive blocks without a source keep their content."""
    offsets = [tuple(int(x) for x in c) for c in offsets]
    p, s, a2a = int(np.prod(dims)), len(offsets), op == iso.ISO_OP_ALLTOALL
    comm = iso.iso_neighborhood_create_mesh(dims, periodic, offsets)
    src, valid = orc.source_ranks_mesh(dims, periodic, offsets)
    init = iso.iso_neighbor_alltoall_init_layout if a2a else iso.iso_neighbor_allgather_init_layout
    for m in sizes + (7,):
        send = torch.randint(0, 256, (p, s if a2a else 1, m), dtype=torch.uint8, device=DEV, generator=torch.Generator(DEV).manual_seed(m))
        for layout in (RANK, SLOT):
            for alg in (BYDIM, iso.ISO_ALG_SX_FUSED):
                given = send.permute(1, 0, 2).contiguous() if layout == SLOT and a2a else send
                recv = torch.full((p * s * m,), 0xEE, dtype=torch.uint8, device=DEV)
                work = torch.full((max(1, iso.iso_workspace_bytes(comm, op, alg, m)),), 0xDD, dtype=torch.uint8, device=DEV)
                req = init(given, recv, m, layout, work, comm, alg)
                start_both_ways(req, recv, work, starts=2)
                iso.iso_request_free(req)
                got = recv.view(s, p, m) if layout == SLOT else recv.view(p, s, m).permute(1, 0, 2)
                for i in range(s):
                    v = torch.from_numpy(np.ascontiguousarray(valid[:, i])).to(DEV)
                    at = torch.from_numpy(np.where(valid[:, i], src[:, i], 0).astype(np.int64)).to(DEV)
                    want = send[:, i if a2a else 0].index_select(0, at)
                    want[~v] = 0xEE
                    assert torch.equal(got[i], want), (dims, m, layout, alg, i)


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("dims,offsets,sizes", [
    ((21, 20, 19), gen.moore(3, 1), gen.stencil_block_sizes(gen.moore(3, 1), 51)), ((33, 31), gen.moore(2, 1), gen.stencil_block_sizes(gen.moore(2, 1), 37)),
    ((9, 8, 7, 6), gen.moore(4, 1), gen.stencil_block_sizes(gen.moore(4, 1), 7)), ((5, 4, 3, 4, 5), gen.moore(5, 1), gen.stencil_block_sizes(gen.moore(5, 1), 3)),
    ((2, 3, 1, 29, 31), gen.random_distinct(5, -3, 3, 30, 6), [(1, 2, 3, 4, 7, 8, 15, 16, 17, 33, 127, 128, 129, 640, 0)[i % 15] for i in range(30)]),
    ((17, 18, 19), gen.moore(3, 1) + [(0, 0, 0), (1, 1, 1), (2, 0, -1)], [(300, 5, 0, 128, 129)[i % 5] for i in range(29)]),
    ((17, 18, 19), gen.moore(3, 1), [200 if i % 2 else 300 for i in range(26)])])                     # no small ones
def test_unequal_blocks_through_all_hops(dims, offsets, sizes, box):
    """Every unit width, blocks of one size among others and empty ones, packed rows and rows with gaps, against the oracle."""
    offsets = [tuple(int(x) for x in c) for c in offsets]
    p, s, sizes = int(np.prod(dims)), len(offsets), [int(x) for x in sizes]
    periodic = [0 if box and j != 1 else 1 for j in range(len(dims))]
    comm = iso.iso_neighborhood_create_mesh(dims, periodic, offsets)
    src, valid = orc.source_ranks_mesh(dims, periodic, offsets)
    src = torch.from_numpy(np.where(valid, src, 0).astype(np.int64)).to(DEV)
    valid = torch.from_numpy(np.ascontiguousarray(valid)).to(DEV)
    for align in (1, 16):
        displs, row = gen.packed_displacements(sizes, align)
        send = torch.randint(0, 256, (p, row), dtype=torch.uint8, device=DEV, generator=torch.Generator(DEV).manual_seed(align))
        for alg in (COMBINED, BYDIM):
            recv = torch.full((p, row), 0xEE, dtype=torch.uint8, device=DEV)
            work = torch.full((max(1, iso.iso_workspace_bytes_v(comm, iso.ISO_OP_ALLTOALL, alg, sizes)),), 0xDD, dtype=torch.uint8, device=DEV)
            req = iso.iso_neighbor_alltoallv_init(send, sizes, displs, row, recv, sizes, displs, row, work, comm, alg)
            start_both_ways(req, recv, work, starts=2)
            iso.iso_request_free(req)
            want = torch.full((p, row), 0xEE, dtype=torch.uint8, device=DEV)
            for i, (at, m) in enumerate(zip(displs, sizes)):
                want[valid[:, i], at:at + m] = send[:, at:at + m].index_select(0, src[valid[:, i], i])
            assert torch.equal(recv, want), (dims, align, alg)


def _from(dims, periodic, vector):
    """For every rank the one `vector` back, and whether there is one, on the device."""
    src, valid = orc.source_ranks_mesh(dims, periodic, [vector])
    return (torch.from_numpy(np.where(valid[:, 0], src[:, 0], 0).astype(np.int64)).to(DEV),
            torch.from_numpy(np.ascontiguousarray(valid[:, 0])).to(DEV))


def _check_workspace(dims, periodic, offsets, op, alg, sizes, layout=RANK):
    """What a start of one launch through all hops leaves in the workspace: of an all-to-all, at every rank on a block's way,
    what the block is there after one of its hops (of two hops there is one such place for a rank); of an allgather, every trie
    node's block, or that of one of the nodes that share a place; everything else, and the bytes around it, untouched."""
    offsets, sizes = [tuple(int(x) for x in c) for c in offsets], [int(x) for x in sizes]
    p, s, d, a2a = int(np.prod(dims)), len(offsets), len(dims), op == iso.ISO_OP_ALLTOALL
    comm = iso.iso_neighborhood_create_mesh(dims, periodic, offsets) if not all(periodic) else iso.iso_neighborhood_create(dims, offsets)
    n_work = iso.iso_workspace_bytes_v(comm, op, alg, sizes)
    store = torch.full((n_work + 512,), 0xDD, dtype=torch.uint8, device=DEV)
    gener = torch.Generator(DEV).manual_seed(p)
    blocks = [torch.randint(0, 256, (p, m), dtype=torch.uint8, device=DEV, generator=gener) for m in (sizes if a2a else sizes[:1])]
    if len(set(sizes)) == 1:
        send = (torch.stack(blocks) if layout == SLOT else torch.cat(blocks, 1)).contiguous()
        recv = torch.empty(p * sum(sizes), dtype=torch.uint8, device=DEV)
        init = iso.iso_neighbor_alltoall_init_layout if a2a else iso.iso_neighbor_allgather_init_layout
        req = init(send, recv, sizes[0], layout, store[256:256 + n_work], comm, alg)
    else:
        displs, row = gen.packed_displacements(sizes, 1)
        send, recv = torch.cat(blocks, 1).contiguous(), torch.empty(p * row, dtype=torch.uint8, device=DEV)
        req = iso.iso_neighbor_alltoallv_init(send, sizes, displs, row, recv, sizes, displs, row, store[256:256 + n_work], comm, alg)
    start, plan = iso.iso_request_start_info(req), iso.iso_request_plan(req)
    assert start["bytes_read"] == (p * sum(sizes) if a2a else start["kernels"] * p * sizes[0])          # the send buffer alone
    info = iso.iso_plan_info(plan)
    entries = [e for q in range(info["launches"]) for e in iso.iso_plan_entries(plan, q)]
    iso.iso_start(req)
    iso.iso_wait(req)
    iso.iso_request_free(req)
    slot_size, states = {}, {}                                    # states: slot -> [(block, source ranks, where)]
    hops, way = {}, {}
    for e in entries:
        if e["dst_buf"] == iso.ISO_BUF_WORK:
            slot_size[e["dst_slot"]] = max(slot_size.get(e["dst_slot"], 0), sizes[e["neighbor"]] if a2a else sizes[0])
        if a2a and sizes[e["neighbor"]]:
            hops.setdefault(e["neighbor"], []).append(e["dim"])
            if e["dst_buf"] == iso.ISO_BUF_WORK:
                way[e["neighbor"]] = e["dst_slot"]
        elif not a2a and e["dst_buf"] == iso.ISO_BUF_WORK:
            routed = list(info["dim_order"])[:list(info["dim_order"]).index(e["dim"]) + 1]
            src, valid = _from(dims, periodic, [offsets[e["ref"]][j] if j in routed else 0 for j in range(d)])
            states.setdefault(e["dst_slot"], []).append((blocks[0], src, valid))
    for i, along in hops.items():
        for t in range(1, len(along)):
            src, valid = _from(dims, periodic, [offsets[i][j] if j in along[:t] else 0 for j in range(d)])
            _, onward = _from(dims, periodic, [-offsets[i][j] if j in along[t:] else 0 for j in range(d)])
            states.setdefault(way[i], []).append((blocks[i], src, valid & onward))
    checked, at = 0, 256
    for slot in range(info["work_slots"]):
        m = slot_size[slot]
        plane = store[at:at + p * m].view(p, m)
        held, due = torch.zeros((p, m), dtype=torch.bool, device=DEV), torch.zeros(p, dtype=torch.bool, device=DEV)
        for block, src, where in states.get(slot, []):
            held |= where[:, None] & (plane == block.index_select(0, src))      # (stores to one place have no order, unit by unit)
            due |= where
            checked += 1
        ok = torch.where(due, held.all(1), (plane == 0xDD).all(1))
        assert bool(ok.all()), (dims, slot, int((~ok).sum()))
        end = at + -(-p * m // 16) * 16
        assert bool((store[at + p * m:end] == 0xDD).all())
        at = end
    assert checked and at == 256 + n_work and bool((store[:256] == 0xDD).all()) and bool((store[at:] == 0xDD).all())


@pytest.mark.parametrize("dims,periodic,offsets,sizes,alg,layout", [
    ((23, 24, 25), (1, 1, 1), gen.moore(3, 1), [128] * 26, COMBINED, RANK),                           # two hops, and three
    ((12, 11, 13), (1, 1, 1), gen.moore(3, 1), [1027] * 26, COMBINED, RANK),
    ((61, 67), (1, 1), gen.moore(2, 2) + [(0, 0), (1, 2), (1, 2)], [1024] * 27, COMBINED, RANK),       # one block per wavefront
    ((7, 6, 5, 8, 9), (1,) * 5, gen.random_distinct(5, -3, 3, 40, 5), [144] * 40, BYDIM, SLOT),
    ((7, 6, 5, 8, 9), (1,) * 5, gen.random_distinct(5, -3, 3, 40, 5), [1024] * 40, COMBINED, RANK),
    ((25, 24, 26), (0, 1, 0), gen.moore(3, 1) + [(25, 0, 1), (2, 25, -2)], [256] * 28, BYDIM, RANK),
    ((7, 6, 9, 5, 8), (1, 0, 0, 1, 0), gen.random_distinct(5, -3, 3, 40, 5), [2048] * 40, BYDIM, SLOT),
    ((21, 20, 19), (1, 1, 1), gen.moore(3, 1), gen.stencil_block_sizes(gen.moore(3, 1), 51), COMBINED, RANK),
    ((13, 12, 11), (0, 1, 0), gen.moore(3, 1), gen.stencil_block_sizes(gen.moore(3, 1), 20), COMBINED, RANK),
    ((5, 4, 3, 4, 5), (1,) * 5, gen.moore(5, 1)[:128], [(1, 2, 4, 8, 16, 64)[i % 6] for i in range(128)], COMBINED, RANK)])
def test_alltoall_stops(dims, periodic, offsets, sizes, alg, layout):
    _check_workspace(dims, periodic, offsets, iso.ISO_OP_ALLTOALL, alg, sizes, layout)


@pytest.mark.parametrize("dims,periodic,offsets,m,alg,layout", [
    ((23, 24, 25), (1, 1, 1), gen.random_distinct(3, -3, 3, 20, 5), 1000, COMBINED, RANK),
    ((7, 6, 5, 8, 9), (1,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 128, COMBINED, RANK),              # pull
    ((8, 9, 8, 7, 5), (1,) * 5, gen.random_distinct(5, -3, 3, 36, 7), 1152, COMBINED, RANK),             # push
    ((9, 8, 8, 9, 8), (1,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 17, COMBINED, RANK),               # plain stores
    ((9, 8, 7, 11), (1,) * 4, gen.random_distinct(4, -3, 3, 30, 5), 100, COMBINED, SLOT),
    ((25, 24, 26), (0, 1, 0), gen.random_distinct(3, -3, 3, 20, 5), 640, BYDIM, RANK)])
def test_allgather_nodes_in_the_workspace(dims, periodic, offsets, m, alg, layout):
    _check_workspace(dims, periodic, offsets, iso.ISO_OP_ALLGATHER, alg, [m] * len(offsets), layout)


@pytest.mark.parametrize("dims,offsets,sizes", [
    ((17, 19), gen.moore(2, 10), [4 + 4 * (i % 2) for i in range(440)]), ((7, 8, 9), gen.moore(3, 3), [(1, 3, 40, 128, 700)[i % 5] for i in range(342)]),
    ((5, 4, 6, 5), gen.moore(4, 1) + gen.von_neumann(4, 2), [(2, 16)[i % 2] for i in range(120)]), ((6, 5, 5), gen.moore(3, 3)[:130], [(8, 4)[i > 0] for i in range(130)])])
def test_unequal_blocks_of_many_neighbours(dims, offsets, sizes):
    """More blocks of a size than one launch takes."""
    offsets = [tuple(int(x) for x in c) for c in offsets]
    comm, p = iso.iso_neighborhood_create(dims, offsets), int(np.prod(dims))
    src, _ = orc.source_ranks_mesh(dims, [1] * len(dims), offsets)
    src = torch.from_numpy(src.astype(np.int64)).to(DEV)
    displs, row = gen.packed_displacements(sizes, 1)
    send = torch.randint(0, 256, (p, row), dtype=torch.uint8, device=DEV, generator=torch.Generator(DEV).manual_seed(p))
    recv = torch.full((p, row), 0xEE, dtype=torch.uint8, device=DEV)
    n_work = iso.iso_workspace_bytes_v(comm, iso.ISO_OP_ALLTOALL, COMBINED, sizes)
    store = torch.full((n_work + 512,), 0xCC, dtype=torch.uint8, device=DEV)
    work = store[256:256 + n_work]
    req = iso.iso_neighbor_alltoallv_init(send, sizes, displs, row, recv, sizes, displs, row, work, comm, COMBINED)
    start_both_ways(req, recv, work, starts=2)
    iso.iso_request_free(req)
    for i, (at, m) in enumerate(zip(displs, sizes)):
        assert torch.equal(recv[:, at:at + m], send[:, at:at + m].index_select(0, src[:, i])), i
    assert bool((store[:256] == 0xCC).all()) and bool((store[256 + n_work:] == 0xCC).all())


@pytest.mark.parametrize("dims,offsets", [
    ((5, 4, 7), gen.moore(3, 1)), ((23, 2, 31), gen.moore(3, 2)), ((17, 1, 19), gen.random_distinct(3, -3, 3, 40, 3)),
    ((6, 7, 5, 9), gen.random_distinct(4, -3, 3, 30, 5)), ((4, 5, 3, 4, 6), gen.random_distinct(5, -3, 3, 40, 5)),
    ((40, 41, 39), [(1, 0, 1), (0, 1, 1), (1, 1, 0), (2, 1, 3), (1, 1, 1), (1, 1, 1), (0, 0, 0)])])
def test_staged_rounds_of_two_dimensions(dims, offsets):
    """One and several hops before the last, along either dimension or both, sides of 1 and 2, repeated neighbours."""
    offsets = [tuple(int(x) for x in c) for c in offsets]
    for m in (16, 48, 256):
        check_exchange(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, m, RANK, send_off=3, recv_off=1)
    check_exchange((64, 65, 66), gen.moore(3, 1), iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, 9, RANK)      # last units that overlap


@pytest.mark.parametrize("dims,n,m", [((7, 8, 7, 8, 8), 40, 208), ((8, 7, 9, 8, 7), 40, 121), ((13, 14, 12, 13), 30, 177)])
def test_large_tiles_of_the_first_two_staged_rounds(dims, n, m):
    """Few ranks of a small tile would end inside a sector: whole units and last units that overlap."""
    offsets = [tuple(int(x) for x in c) for c in gen.random_distinct(len(dims), -3, 3, n, 160607676)]
    check_exchange(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, m, RANK, send_off=3, recv_off=1)
