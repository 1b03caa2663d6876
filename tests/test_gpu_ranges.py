"""iso_start takes the rounds of one dimension of ISO_ALG_COMBINED together; iso_start_range still runs the
schedule round by round.  Both against the oracle, every byte: equal blocks in both layouts (wide, ragged and
narrow units, blocks taken in groups of ranks), unequal blocks, a mesh with a periodic dimension."""
import numpy as np
import pytest
import torch

import iso_inputs as gen
import paper_1606_07676_amd as iso
from oracle import iso_oracle as orc

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
CASES = [((6, 5), gen.von_neumann(2, 2)), ((7, 5, 6), gen.moore(3, 1)), ((13, 11, 9), gen.moore(3, 1)),
         ((4, 3, 5, 4), gen.random_distinct(4, -3, 3, 30, 3)), ((3, 4, 2, 5, 3), gen.random_distinct(5, -3, 3, 150, 4))]


def _both_ways(req, recv, want):
    n = iso.iso_request_info(req)["launches"]
    for by_rounds in (False, True, False):
        recv.fill_(0xEE)
        if by_rounds:
            for q in range(n):
                iso.iso_start_range(req, q, 1)
        else:
            iso.iso_start(req)
        iso.iso_wait(req)
        got = recv.cpu().numpy().reshape(want.shape)
        assert np.array_equal(got, want), ("rounds" if by_rounds else "start", got.shape)
    iso.iso_request_free(req)


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_equal_blocks(case, op):
    dims, offsets = CASES[case]
    p, s = int(np.prod(dims)), len(offsets)
    comm = iso.iso_neighborhood_create(dims, np.asarray(offsets, np.int32).reshape(s, len(dims)))
    a2a = op == iso.ISO_OP_ALLTOALL
    for m in (3, 16, 200, 1024, 2064):
        send_h = gen.alltoall_send(50 + case, p, s, m) if a2a else gen.allgather_send(50 + case, p, m)
        want = (orc.alltoall if a2a else orc.allgather)(dims, offsets, send_h)
        for layout in (iso.ISO_LAYOUT_RANK_MAJOR, iso.ISO_LAYOUT_SLOT_MAJOR):
            slot = layout == iso.ISO_LAYOUT_SLOT_MAJOR
            host = np.ascontiguousarray(send_h.transpose(1, 0, 2)) if slot and a2a else send_h
            send = torch.from_numpy(host).to(DEV)
            recv = torch.empty(p * s * m, dtype=torch.uint8, device=DEV)
            work = torch.empty(max(1, iso.iso_workspace_bytes(comm, op, iso.ISO_ALG_COMBINED, m)), dtype=torch.uint8,
                               device=DEV)
            init = iso.iso_neighbor_alltoall_init_layout if a2a else iso.iso_neighbor_allgather_init_layout
            _both_ways(init(send, recv, m, layout, work, comm, iso.ISO_ALG_COMBINED), recv,
                       np.ascontiguousarray(want.transpose(1, 0, 2)) if slot else want)


@pytest.mark.parametrize("case", range(3))
def test_unequal_blocks(case):
    dims, offsets = CASES[case]
    p, s = int(np.prod(dims)), len(offsets)
    comm = iso.iso_neighborhood_create(dims, np.asarray(offsets, np.int32).reshape(s, len(dims)))
    sizes = gen.stencil_block_sizes(offsets, 9)
    displs, row = gen.packed_displacements(sizes)
    send_h = np.random.default_rng(case).integers(0, 256, (p, row), dtype=np.uint8)
    want = np.full((p, row), 0xEE, np.uint8)
    src = orc.allgather(dims, offsets, np.arange(p, dtype=np.int32).reshape(p, 1).view(np.uint8).copy())
    src = src.reshape(p, s, 4).view(np.int32)[:, :, 0]
    for i in range(s):
        want[:, displs[i]:displs[i] + sizes[i]] = send_h[src[:, i], displs[i]:displs[i] + sizes[i]]
    send = torch.from_numpy(send_h).to(DEV)
    recv = torch.empty(p * row, dtype=torch.uint8, device=DEV)
    work = torch.empty(max(1, iso.iso_workspace_bytes_v(comm, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED, sizes)),
                       dtype=torch.uint8, device=DEV)
    _both_ways(iso.iso_neighbor_alltoallv_init(send, sizes, displs, row, recv, sizes, displs, row, work, comm,
                                               iso.ISO_ALG_COMBINED), recv, want)


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
def test_mesh(op):
    dims, periodic, offsets = (9, 7, 8), [False, True, False], gen.moore(3, 1)
    p, s, m = int(np.prod(dims)), len(offsets), 100
    comm = iso.iso_neighborhood_create_mesh(dims, periodic, np.asarray(offsets, np.int32))
    a2a = op == iso.ISO_OP_ALLTOALL
    send_h = gen.alltoall_send(3, p, s, m) if a2a else gen.allgather_send(3, p, m)
    want = np.full((p, s, m), 0xEE, np.uint8)
    (orc.alltoall_mesh if a2a else orc.allgather_mesh)(dims, periodic, offsets, send_h, want)
    send = torch.from_numpy(send_h).to(DEV)
    recv = torch.empty(p * s * m, dtype=torch.uint8, device=DEV)
    work = torch.empty(max(1, iso.iso_workspace_bytes(comm, op, iso.ISO_ALG_COMBINED, m)), dtype=torch.uint8, device=DEV)
    init = iso.iso_neighbor_alltoall_init if a2a else iso.iso_neighbor_allgather_init
    _both_ways(init(send, recv, m, work, comm, iso.ISO_ALG_COMBINED), recv, want)
