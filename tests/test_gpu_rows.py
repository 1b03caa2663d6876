"""All-to-alls and allgathers whose receive rows are written whole (deliver_bytes_kernel, any block size), and stars in
one launch: at the edges of their tiles against the oracle, in large against the straightforward exchange."""
import numpy as np
import pytest
import torch

import iso_inputs as gen
import paper_1606_07676_amd as iso
from oracle import iso_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 64


def _received(dims, offsets, op, alg, m, send, shift=0, layout=iso.ISO_LAYOUT_RANK_MAJOR):
    """The receive buffer, `shift` bytes off its alignment, between guard bytes that must survive."""
    p, s = int(np.prod(dims)), len(offsets)
    comm = iso.iso_neighborhood_create(dims, offsets)
    store = torch.full((p * s * m + 2 * GUARD + shift,), 0xEE, dtype=torch.uint8, device=DEV)
    recv = store[GUARD + shift:GUARD + shift + p * s * m]
    work = torch.full((max(1, iso.iso_workspace_bytes(comm, op, alg, m)),), 0xDD, dtype=torch.uint8, device=DEV)
    init = iso.iso_neighbor_alltoall_init_layout if op == iso.ISO_OP_ALLTOALL else iso.iso_neighbor_allgather_init_layout
    req = init(send, recv, m, layout, work, comm, alg)
    for _ in range(2):
        iso.iso_start(req)
    iso.iso_wait(req)
    kernels = iso.iso_request_start_info(req)["kernels"]
    iso.iso_request_free(req)
    assert bool((store[:GUARD + shift] == 0xEE).all()) and bool((store[GUARD + shift + p * s * m:] == 0xEE).all()), (dims, m)
    return recv, kernels


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("dims,offsets", [((5, 4, 7), gen.moore(3, 1)), ((37, 11), gen.von_neumann(2, 2)), ((13, 11, 6), gen.random_distinct(3, -3, 3, 20, 5)),
                                          ((2, 3), [(0, 0), (1, 1), (1, 1), (0, 2)]), ((1,), [(0,)]), ((259,), gen.von_neumann(1, 1))])
def test_rows_of_any_block_size(dims, offsets, op):
    """Blocks shorter than a unit, one byte either side of whole units, rows up to the small tile's 16 KiB, up to the
    large one's 32 KiB and just beyond it, fewer ranks than a tile takes, and receive buffers at odd addresses."""
    p, s = int(np.prod(dims)), len(offsets)
    small, fits = (1024 * 16 - 1) // s, (2048 * 16 - 15) // s
    for m in (1, 2, 3, 7, 9, 15, 17, 31, 33, 100, 257, small, fits - 1, fits, fits + 1):
        send_h = gen.alltoall_send(5, p, s, m) if op == iso.ISO_OP_ALLTOALL else gen.allgather_send(5, p, m)
        want = (orc.alltoall if op == iso.ISO_OP_ALLTOALL else orc.allgather)(dims, offsets, send_h).reshape(-1)
        send = torch.from_numpy(send_h).to(DEV)
        for shift in (0, 1, 13):
            got, _ = _received(dims, offsets, op, iso.ISO_ALG_COMBINED_STAGED, m, send, shift)
            assert np.array_equal(got.cpu().numpy(), want), (dims, m, shift)


@pytest.mark.parametrize("dims,offsets,m,alg,layout,kernels", [
    ((24, 24, 24), gen.moore(3, 1), 150, 0, 0, 3), ((23, 24, 27), gen.moore(3, 1), 33, 0, 0, 3), ((67, 63), gen.moore(2, 2), 101, 0, 0, 2),
    ((20, 21, 19), gen.von_neumann(3, 2), 255, 0, 0, 3), ((7, 7, 7, 7), gen.moore(4, 1), 72, 0, 0, 4), ((16, 17, 18), [(0, 0, 0)] + gen.moore(3, 1) + [(1, 1, 1)], 96, 0, 0, 3),
    ((64, 64, 64), gen.moore(3, 1), 16, 0, 0, 3), ((64, 64, 64), gen.moore(3, 1), 7, 0, 0, 3), ((64, 64, 64), gen.moore(3, 1), 84, 1, 0, 3), ((320, 331), gen.moore(2, 2), 200, 1, 0, 2),
    ((40, 41, 39), gen.von_neumann(3, 1), 20, 0, 0, 1), ((300, 301), gen.von_neumann(2, 1), 100, 0, 1, 1), ((9, 8, 7, 6, 5), gen.von_neumann(5, 1), 300, 0, 0, 1),
    ((50, 51), [(1, 0), (-1, 0), (0, 3), (0, 0), (0, -2), (1, 0)], 17, 0, 0, 1), ((40, 41, 39), gen.von_neumann(3, 1), 2048, 0, 0, 1)])
def test_large_collectives_against_the_straightforward_exchange(dims, offsets, m, alg, layout, kernels):
    p, s = int(np.prod(dims)), len(offsets)
    offsets = [tuple(int(x) for x in c) for c in offsets]
    send = torch.randint(0, 256, (p * s * m,), dtype=torch.uint8, device=DEV, generator=torch.Generator(DEV).manual_seed(3))
    want, _ = _received(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_SX_FUSED, m, send, 0, layout)
    for shift in (0, 5):
        got, n = _received(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m, send, shift, layout)
        assert n == kernels and torch.equal(got, want), (dims, m, shift, n)


@pytest.mark.parametrize("layout", [iso.ISO_LAYOUT_RANK_MAJOR, iso.ISO_LAYOUT_SLOT_MAJOR])
@pytest.mark.parametrize("dims,m", [((40, 41, 39), 20), ((9, 8, 7, 6, 5), 100), ((300, 301), 255)])
def test_star_allgather_in_one_launch(dims, m, layout):
    p, offsets = int(np.prod(dims)), gen.von_neumann(len(dims), 1)
    send = torch.randint(0, 256, (p * m,), dtype=torch.uint8, device=DEV, generator=torch.Generator(DEV).manual_seed(4))
    want, _ = _received(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_SX_ROUNDS, m, send, 0, layout)
    got, n = _received(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_COMBINED, m, send, 0, layout)
    assert n == 1 and torch.equal(got, want)
