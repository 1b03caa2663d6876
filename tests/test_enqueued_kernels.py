"""Which kernels a call enqueues, on the CPU: the library's host code over a stand-in HIP runtime."""
import subprocess
import time

import numpy as np
import pytest

import iso_inputs as gen
import paper_1606_07676_amd as iso

COMBINED = [iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM, iso.ISO_ALG_COMBINED_STAGED]


def _names(kernels):
    return [k.split("<")[0] for k in kernels]


def _noalloc(stub, dims, offsets, m, alg, periodic=None):
    p, s = int(np.prod(dims)), len(offsets)
    comm = stub.comm(dims, offsets, periodic)
    with stub.buffers(p * s * m, p * s * m) as (send, recv):
        return _names(stub.launched(lambda: stub.iso.iso_neighbor_alltoall_noalloc(send, recv, m, comm, alg, 0)))


@pytest.mark.parametrize("alg", COMBINED)
def test_allocation_free_call_of_a_small_alltoall_is_one_kernel(stub_library, alg):
    assert _noalloc(stub_library, (8, 8, 8), gen.moore(3, 1), 64, alg) == ["chain_kernel"]


def test_allocation_free_call_stores_only_tables_that_its_kernels_read(stub_library):
    """Entries, and the residues of the offsets where a kernel reads them (a mesh, more than five dimensions)."""
    for dims, offsets, alg, periodic, want in (
            ((8, 8, 8), gen.moore(3, 1), iso.ISO_ALG_SX_FUSED, None, ["table_store_kernel", "vector_round_kernel"]),
            ((16, 16, 16), gen.von_neumann(3, 1), iso.ISO_ALG_ONEHOP, None,
             ["table_store_kernel"] + 6 * ["shift_round_kernel"]),
            ((2, 3, 2, 3, 2, 4), gen.von_neumann(6, 1), iso.ISO_ALG_SX_FUSED, None,
             2 * ["table_store_kernel"] + ["vector_round_kernel"]),
            ((8, 8), gen.von_neumann(2, 1), iso.ISO_ALG_COMBINED_BYDIM, (0, 0),
             3 * ["table_store_kernel"] + 2 * ["mesh_shift_round_kernel"])):
        assert _noalloc(stub_library, dims, offsets, 64, alg, periodic) == want, dims


def test_allocation_free_calls_on_one_handle_are_those_of_new_handles(stub_library):
    """The handle keeps the schedules that these calls build: every algorithm its own, and what is refused stays refused."""
    niso, dims, offsets, m = stub_library.iso, (9, 4, 7), gen.moore(3, 1), 48
    p, s = int(np.prod(dims)), len(offsets)
    comm = stub_library.comm(dims, offsets)
    with stub_library.buffers(p * s * m, p * s * m) as (send, recv):
        for alg in (0, 1, 2, 3, 4, 5, 0, 5, 3, -1, 6, 2, 1 << 30, 4):
            if alg not in range(6):
                with pytest.raises(niso.IsoError) as e:
                    niso.iso_neighbor_alltoall_noalloc(send, recv, m, comm, alg, 0)
                assert e.value.status == iso.ISO_ERR_ARG
                continue
            got = _names(stub_library.launched(lambda: niso.iso_neighbor_alltoall_noalloc(send, recv, m, comm, alg, 0)))
            assert got == _noalloc(stub_library, dims, offsets, m, alg), alg


def test_allocation_free_call_refuses_the_tables_it_always_refused(stub_library):
    """3900 neighbours in five dimensions: the entries alone would fit the table's 256 KiB, with the residues they do
    not, and the refusal does not depend on whether the kernels read them."""
    offsets = gen.random_distinct(5, -3, 3, 3900, 1)
    assert 3900 * 48 < iso.ISO_NOALLOC_TABLE_BYTES < 3900 * (48 + 20)
    with pytest.raises(stub_library.iso.IsoError) as e:
        _noalloc(stub_library, (2, 2, 2, 2, 2), offsets, 16, iso.ISO_ALG_SX_ROUNDS)
    assert e.value.status == iso.ISO_ERR_SCRATCH


@pytest.mark.parametrize("dims,offsets,m,stores,rounds", [
    ((1200000, 64), [(0, 1), (0, -1)], 1, 27, 1), ((400, 400, 400), gen.von_neumann(3, 1), 1, 64, 3),
    ((64, 64, 64), gen.von_neumann(3, 1), 256, 6, 3), ((64, 64, 64), gen.von_neumann(3, 1), 64, 3, 3),
    ((262144, 16), gen.von_neumann(2, 1), 16, 5, 2), ((12, 12, 12), gen.moore(3, 1), 40, 3, 3)])
def test_allocation_free_call_on_boxes_stores_bitmaps_by_the_tile(stub_library, dims, offsets, m, stores, rounds):
    """The bitmaps of a mesh share the table with the entries and the residues, and every 3 KiB of it is a launch: as many
    as with a bit per tile of 256 units, and none refused that fits so."""
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        names = _noalloc(stub_library, dims, offsets, m, alg, (0,) * len(dims))
        assert names == stores * ["table_store_kernel"] + rounds * ["mesh_shift_round_kernel"], (alg, len(names))


@pytest.mark.parametrize("dims,offsets,m,kernels", [
    ((8, 8, 8), gen.von_neumann(3, 1), 60, "chain"), ((16, 16), gen.von_neumann(2, 1), 100, "chain"), ((6, 6, 4, 6), gen.von_neumann(4, 2), 93, "chain"),
    ((700,), [(1,), (-1,), (3,)], 11, "store deliver_bytes"), ((50,), [(0,), (2,), (-1,)], 1, "chain"), ((1, 1), gen.moore(2, 1), 35, "store deliver_bytes"),
    ((15, 19, 16), [(-2, 0, -3), (3, 0, 2)], 3, "store shift_round deliver_bytes"),
    ((9, 6, 12), gen.moore(3, 2), 86, "store store store store store store shift_round shift_round deliver_bytes"),
    ((8, 8, 8), gen.von_neumann(3, 1), 64, "store deliver"), ((32, 32, 32), gen.von_neumann(3, 1), 100, "store deliver_bytes")])
def test_allocation_free_call_of_the_staged_schedule(stub_library, dims, offsets, m, kernels):
    """Rows of any block size cost a launch for their records there: the chain stands against a launch per dimension, and
    nothing is stored that no kernel reads."""
    names = _noalloc(stub_library, dims, offsets, m, iso.ISO_ALG_COMBINED_STAGED)
    assert " ".join(n.replace("_kernel", "").replace("table_", "") for n in names) == kernels


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("dims,offsets,m,kernels", [
    ((8, 8), gen.moore(2, 1), 64, 1), ((8, 8, 8), gen.moore(3, 1), 64, 1), ((32, 32), gen.von_neumann(2, 2), 64, 1),
    ((8, 8), [(1, 1), (0, 1), (2, 0)], 2056, 1), ((4, 3), [(1, 1), (1, 1), (0, 0), (0, 0), (5, -7), (2, 0)], 5464, 1),
    ((5, 5, 5, 5), gen.von_neumann(4, 1), 1000, 1), ((5, 5, 5, 5), gen.von_neumann(4, 1), 2000, 4),
    ((16, 16), gen.von_neumann(2, 1), 3000, 1), ((16, 16), gen.von_neumann(2, 1), 5000, 2), ((45, 45), gen.von_neumann(2, 1), 256, 2), ((16, 16), gen.moore(2, 1), 400, 1),
    ((32, 32), gen.moore(2, 1), 100, 2), ((10, 10, 10), gen.moore(3, 1), 16, 1), ((10, 10, 10), gen.moore(3, 1), 64, 1),
    ((16, 16), gen.von_neumann(2, 2), 400, 1), ((16, 16), gen.von_neumann(2, 2), 1000, 2),
    ((11, 11, 11), gen.moore(3, 1), 16, 3), ((12, 12, 12), gen.moore(3, 1), 32, 3), ((12, 12, 12), gen.von_neumann(3, 1), 400, 3),
    ((4096,), gen.von_neumann(1, 1), 16, 1), ((16, 16), gen.moore(2, 1), 1000, 2), ((32, 32), gen.von_neumann(2, 2), 300, 2),
    ((8, 8, 8), gen.moore(3, 1), 200, 3), ((10, 10, 10), gen.moore(3, 1), 100, 3)])
def test_small_collectives_take_one_launch_where_it_saves_enough(stub_library, dims, offsets, m, kernels, op):
    """The chain kernel's limit is per launch saved: none for a schedule of one launch."""
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        names = _names(stub_library.start(dims, offsets, op, alg, m))
        chained = kernels == 1 and len(dims) > 1
        assert names == ["chain_kernel"] if chained else (len(names) == kernels and "chain_kernel" not in names), (alg, names)


@pytest.mark.parametrize("dims,offsets,m,kernels", [
    ((8, 8, 8), gen.moore(3, 2), 64, 1), ((11, 11, 11), gen.moore(3, 2), 64, 3), ((4, 4, 4, 4), gen.moore(4, 1), 200, 1), ((4, 4, 4, 4), gen.moore(4, 1), 600, 4),
    ((7, 7, 7, 7), gen.random_distinct(4, -3, 3, 30, 5), 16, 4), ((8, 8, 8, 8), gen.random_distinct(4, -3, 3, 30, 5), 16, 4), ((2, 2, 2, 2, 2), gen.moore(5, 2), 16, 6)])
def test_many_chains_fill_the_chip_with_more(stub_library, dims, offsets, m, kernels):
    """Chains of several hops in 64 workgroups and more go further; the allocation-free call carries 72 hops at most."""
    names = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED, m))
    assert len(names) == kernels and ("chain_kernel" in names) == (kernels == 1), names
    if kernels == 1:
        assert "chain_kernel" not in _noalloc(stub_library, dims, offsets, m, iso.ISO_ALG_COMBINED)


@pytest.mark.parametrize("dims,offsets,m,kernels", [
    ((20, 16), gen.moore(2, 2), 586, 2), ((13, 13), gen.von_neumann(2, 2), 2784, 2), ((13, 16), gen.moore(2, 2), 796, 2), ((13, 16), gen.moore(2, 2), 64, 1),
    ((5, 5, 5), gen.moore(3, 2), 240, 1)])
def test_more_sectors_only_where_two_launches_are_saved(stub_library, dims, offsets, m, kernels):
    """A chain that replaces two launches keeps 48 Ki sectors, however many workgroups share them; the allocation-free call
    saves the launch of its table as well (up to 72 hops)."""
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        names = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m))
        assert len(names) == kernels and ("chain_kernel" in names) == (kernels == 1), (alg, names)
        assert _noalloc(stub_library, dims, offsets, m, alg)[-1] == ("chain_kernel" if len(dims) == 2 else "shift_round_kernel")


@pytest.mark.parametrize("dims,offsets,m,width", [((5, 4, 7, 6, 4), gen.von_neumann(5, 1), 6, "unsigned short, false"),
                                                  ((13, 14, 15), gen.von_neumann(3, 1), 5, "unsigned char, false"),
                                                  ((46, 47), gen.von_neumann(2, 1), 3, "unsigned char, false"),
                                                  ((45, 45), gen.von_neumann(2, 1), 6, "unsigned int, true")])
def test_columns_of_one_unit_take_units_that_divide_the_block(stub_library, dims, offsets, m, width):
    for op in (iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER):
        (kernel,) = stub_library.start(dims, offsets, op, iso.ISO_ALG_COMBINED, m)
        assert kernel.startswith(f"chain_kernel<{width}"), kernel


# cache policies: 0 cached loads, streaming stores; 1 streaming both; 2 cached, plain stores; 3 streaming loads, plain stores;
# 4 by the block's size
POLICY_ARGUMENT = {"shift_round_kernel": 2, "mesh_shift_round_kernel": 2, "shift_round_uniform_kernel": 0,
                   "staged_round_kernel": 1, "deliver_kernel": 1, "block_round_kernel": 2, "vector_round_kernel": 3,
                   "vector_round_uniform_kernel": 1, "deliver_bytes_kernel": 1}
NO_POLICY = {"chain_kernel", "shift_push_kernel", "push_round_kernel"}


def _policies(kernels):
    out = set()
    for k in kernels:
        name, args = k.rstrip(">").split("<")
        if name not in NO_POLICY:
            out.add((name.replace("_kernel", "").replace("_round", ""), int(args.split(", ")[POLICY_ARGUMENT[name]])))
    return out


@pytest.mark.parametrize("dims,offsets,m,layout,periodic,want", [
    ((30, 30, 30), gen.von_neumann(3, 1), 1000, 0, None, 0), ((32, 32, 32), gen.moore(3, 1), 200, 0, None, 0),
    ((40, 40, 40), gen.moore(3, 1), 160, 0, (0, 0, 0), 0), ((45, 37, 29), gen.moore(3, 1), 100, 1, (0, 0, 0), 0),
    ((300, 300), gen.moore(2, 2), 56, 0, None, 0), ((24, 24, 24), gen.von_neumann(3, 2), 36, 0, (0, 0, 0), 0),
    ((64, 64, 64), gen.moore(3, 1), 32, 0, None, 2), ((64, 64, 64), gen.moore(3, 1), 56, 0, None, 0),
    ((8, 8, 8, 8, 8), gen.random_distinct(5, -3, 3, 40, 5), 40, 0, None, 2)])
def test_allgather_rounds_stream_their_stores(stub_library, dims, offsets, m, layout, periodic, want):
    """Plain stores only for blocks of less than a sector, rank-major, three and more dimensions, up to the cache."""
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        got = _policies(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, alg, m, layout, periodic))
        assert got == {("mesh_shift" if periodic else "shift", want)}


@pytest.mark.parametrize("dims,offsets,m,layout,periodic,want", [
    ((16, 16, 16), gen.moore(3, 1), 128, 0, None, 1), ((20, 20, 20), gen.moore(3, 1), 64, 0, None, 1),
    ((60, 60), gen.moore(2, 2), 128, 0, None, 1), ((24, 24, 24), gen.moore(3, 1), 64, 1, None, 1),
    ((24, 24, 24), gen.moore(3, 1), 64, 1, (0, 0, 0), 1), ((24, 24, 24), gen.moore(3, 1), 100, 1, None, 1),
    ((100, 100), gen.von_neumann(2, 2), 256, 1, None, 1),
    ((16, 16, 16), gen.moore(3, 1), 64, 0, None, 2), ((60, 60), gen.moore(2, 2), 64, 1, None, 2)])
def test_alltoall_rounds_of_whole_sectors_stream_beyond_8_MiB(stub_library, dims, offsets, m, layout, periodic, want):
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        got = _policies(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m, layout, periodic))
        assert got == {("mesh_shift" if periodic else "shift", want)}


@pytest.mark.parametrize("dims,offsets,m,periodic,want", [
    ((64, 64, 64), gen.moore(3, 1), 20, None, 3), ((64, 64, 64), gen.moore(3, 1), 16, None, 2),
    ((300, 300), gen.moore(2, 2), 25, None, 2), ((100, 100), gen.moore(2, 1), 48, (0, 0), 2),
    ((32, 32, 32), gen.moore(3, 1), 100, None, 2), ((45, 37, 29), gen.moore(3, 1), 100, (0, 0, 0), 2),
    ((16, 16, 16), gen.moore(3, 1), 100, None, 1), ((16, 16, 16), gen.moore(3, 1), 200, (0, 0, 0), 1),
    ((20, 20, 20), gen.moore(3, 1), 100, None, 2),
    ((60, 60), gen.moore(2, 2), 200, None, 1), ((300, 300), gen.von_neumann(2, 1), 100, None, 0),
    ((200, 200), gen.moore(2, 1), 200, None, 0), ((200, 200), gen.moore(2, 1), 100, (0, 0), 1),
    ((16, 16, 16), gen.moore(3, 1), 400, None, 0), ((100, 100), gen.moore(2, 2), 300, None, 0),
    ((12, 12, 12), gen.moore(3, 1), 600, None, 1), ((30, 30, 30), gen.von_neumann(3, 1), 1000, None, 0),
    ((30, 30, 30), gen.von_neumann(3, 1), 1000, (0, 0, 0), 1), ((32, 32, 32), gen.moore(3, 1), 300, None, 3),
    ((50, 50, 50), gen.von_neumann(3, 1), 200, None, 0), ((300, 300), gen.von_neumann(2, 1), 400, None, 0),
    ((64, 64, 64), gen.von_neumann(3, 1), 140, (0, 0, 0), 0), ((100, 100, 100), gen.von_neumann(3, 1), 36, None, 3),
    ((32, 32, 32), gen.moore(3, 1), 500, None, 1), ((64, 64, 64), gen.moore(3, 1), 48, None, 1)])
def test_alltoall_rounds_of_part_sectors(stub_library, dims, offsets, m, periodic, want):
    """By block size, hops per block, and size of the collective against the last-level cache."""
    got = _policies(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_BYDIM, m, 0, periodic))
    assert got == {("mesh_shift" if periodic else "shift", want)}


@pytest.mark.parametrize("dims,offsets,m", [((64, 64, 64), gen.moore(3, 1), 16), ((64, 64, 64), gen.von_neumann(3, 1), 64),
                                            ((32, 32, 32), gen.moore(3, 1), 128)])
def test_staged_allgather_streams_its_stores(stub_library, dims, offsets, m):
    got = _policies(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_COMBINED_STAGED, m))
    assert ("deliver", 0) in got and all(policy == 0 for _, policy in got)


@pytest.mark.parametrize("dims,offsets,m,rounds,last", [
    ((64, 64, 64), gen.moore(3, 1), 16, 2, 0), ((20, 20, 20), gen.moore(3, 1), 64, 1, 1), ((32, 32, 32), gen.moore(3, 1), 32, 1, 1),
    ((44, 44, 44), gen.moore(3, 1), 32, 2, 0), ((9, 9, 9, 9), gen.moore(4, 1), 176, 2, 0),
    ((18, 18, 18), gen.moore(3, 1), 240, 1, 1), ((40, 40, 40), gen.moore(3, 1), 64, 0, 0), ((64, 64, 64), gen.moore(3, 1), 32, 0, 1),
    ((32, 32, 32), gen.moore(3, 1), 128, 1, 1), ((20, 20, 20), gen.moore(3, 1), 256, 1, 1), ((64, 64, 64), gen.moore(3, 1), 80, 1, 1)])
def test_staged_alltoall_by_block_size_and_size(stub_library, dims, offsets, m, rounds, last):
    got = _policies(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, m))
    assert {("staged", rounds), ("deliver", last)} <= got <= {("staged", rounds), ("deliver", last), ("shift", 1)}


def test_staged_rounds_between_planes_stream(stub_library):
    offsets = gen.random_distinct(5, -3, 3, 40, 5)
    got = _policies(stub_library.start((6, 6, 6, 6, 6), offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, 48))
    assert ("shift", 1) in got and all(policy == 1 for _, policy in got)


@pytest.mark.parametrize("dims,offsets,m,alg,want", [
    ((24, 24, 24), gen.moore(3, 1), 100, 0, ["staged_round_kernel"] * 2 + ["deliver_bytes_kernel"]), ((24, 24, 24), gen.moore(3, 1), 20, 0, ["shift_round_kernel"] * 3),
    ((64, 64, 64), gen.moore(3, 1), 20, 0, ["staged_round_kernel"] * 2 + ["deliver_bytes_kernel"]), ((64, 64, 64), gen.moore(3, 1), 192, 0, ["shift_round_kernel"] * 3),
    ((64, 64, 64), gen.moore(3, 1), 100, 1, ["staged_round_kernel"] * 2 + ["deliver_bytes_kernel"]), ((32, 32, 32), gen.moore(3, 1), 200, 1, ["shift_round_kernel"] * 3),
    ((20, 20, 20), gen.moore(3, 2), 264, 0, ["shift_round_kernel"] * 3), ((100, 100), gen.moore(2, 1), 500, 0, ["staged_round_kernel", "deliver_bytes_kernel"]),
    ((24, 24, 24), gen.von_neumann(3, 1), 100, 0, ["vector_round_kernel"]), ((24, 24, 24), gen.von_neumann(3, 1), 100, 1, ["shift_round_kernel"] * 3),
    ((24, 24, 24), gen.von_neumann(3, 1), 300, 0, ["vector_round_kernel"]), ((250000,), gen.von_neumann(1, 1), 256, 0, ["shift_round_kernel"])])
def test_alltoalls_that_write_rows_whole_or_all_at_once(stub_library, dims, offsets, m, alg, want):
    names = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m))
    assert names == want
    listed = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m, by_rounds=True))
    assert "deliver_bytes_kernel" not in listed and "vector_round_kernel" not in listed


@pytest.mark.parametrize("dims,m,rounds,last", [
    ((24, 24, 24), 100, 2, 0), ((29, 29, 29), 105, 2, 0), ((29, 29, 29), 106, 3, 0), ((40, 40, 40), 79, 3, 0), ((40, 40, 40), 81, 3, 1), ((64, 64, 64), 100, 3, 1), ((64, 64, 64), 15, 0, 0)])
def test_cache_policy_of_rows_of_any_block_size(stub_library, dims, m, rounds, last):
    """26 neighbours.  The rounds in front of the rows stream their loads above a quarter of the cache, the rows both above
    half of it; narrower units have one form."""
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_STAGED):
        got = _policies(stub_library.start(dims, gen.moore(3, 1), iso.ISO_OP_ALLTOALL, alg, m))
        got.discard(("shift", rounds))                       # the staged schedule's small blocks keep the plain kernel
        assert got <= {("staged", rounds), ("deliver_bytes", last)} and ("deliver_bytes", last) in got, (alg, got)


@pytest.mark.parametrize("dims,offsets,alg,rows", [
    ((600, 600), gen.moore(2, 1), 0, False), ((420, 420), gen.von_neumann(2, 2), 0, False), ((300, 300), gen.moore(2, 2), 0, True),
    ((662, 503), gen.random_distinct(2, -3, 3, 10, 5), 0, True), ((600, 600), gen.random_distinct(2, -3, 3, 8, 5), 0, True), ((64, 64, 64), gen.moore(3, 1), 0, True), ((24, 24, 24), gen.moore(3, 1), 0, False),
    ((80, 80, 80), gen.von_neumann(3, 2), 1, True), ((16, 16, 16, 16), gen.moore(4, 1), 0, True), ((20, 20, 20, 20), gen.moore(4, 1), 0, False),
    ((20, 20, 20, 20), gen.moore(4, 1), 1, False), ((12,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 0, False)])
def test_rows_of_64_byte_blocks(stub_library, dims, offsets, alg, rows):
    """Half a line: from 48 MiB on, in two dimensions from eight hops to five blocks, in four and more up to 384 MiB."""
    names = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, 64))
    assert names == (["staged_round_kernel"] * (len(dims) - 1) + ["deliver_bytes_kernel"] if rows else ["shift_round_kernel"] * len(dims))


@pytest.mark.parametrize("s,m,small", [(4, 4095, False), (8, 2047, False), (1, 16383, False), (1, 16369, True), (4, 4092, True), (16, 1023, True)])
def test_rows_next_to_a_small_tile(stub_library, s, m, small):
    """A tile by bytes holds up to 15 bytes more than the rows: the alignment of the receive buffer."""
    for op in (iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER):
        kernels = stub_library.start((64, 65), [(i + 1, 1) for i in range(s)], op, iso.ISO_ALG_COMBINED_STAGED, m)
        (last,) = [k for k in kernels if k.startswith("deliver_bytes_kernel")]
        assert last.endswith("4u>" if small else "8u>"), kernels


@pytest.mark.parametrize("op,m,want", [(iso.ISO_OP_ALLTOALL, 200, 0), (iso.ISO_OP_ALLTOALL, 100, 1), (iso.ISO_OP_ALLTOALL, 40, 2),
                                       (iso.ISO_OP_ALLGATHER, 40, 0)])
def test_staged_schedule_on_the_general_kernels(stub_library, op, m, want):
    """Blocks that are no multiple of 16 bytes: the rounds that read or write rows."""
    got = _policies(stub_library.start((20, 20, 20), gen.moore(3, 1), op, iso.ISO_ALG_COMBINED_STAGED, m))
    assert ("shift", want) in got


@pytest.mark.parametrize("dims,sizes,periodic,want", [
    ((40, 40, 40), [256 - i % 2 for i in range(26)], None, 1), ((40, 40, 40), [256 - i % 2 for i in range(26)], (0, 0, 0), 1),
    ((16, 16, 16), [64 - i % 2 for i in range(26)], None, 1), ((20, 20, 20), [256 - i % 2 for i in range(26)], None, 0),
    ((20, 20, 20), gen.stencil_block_sizes(gen.moore(3, 1), 25), None, 0),
    ((24, 24, 24), gen.stencil_block_sizes(gen.moore(3, 1), 20), None, 0),
    ((64, 64, 64), gen.stencil_block_sizes(gen.moore(3, 1), 4), None, 2),
    ((32, 32, 32), gen.stencil_block_sizes(gen.moore(3, 1), 9), (0, 0, 0), 2),
    ((64, 64, 64), gen.stencil_block_sizes(gen.moore(3, 1), 9), None, 0)])
def test_rounds_of_unequal_blocks(stub_library, dims, sizes, periodic, want):
    """Streaming loads where all blocks have the same number of units, plain stores for small blocks near the cache."""
    got = _policies(stub_library.start_unequal(dims, gen.moore(3, 1), iso.ISO_ALG_COMBINED_BYDIM, list(sizes), periodic))
    assert got == {("block", want)}


FIVE = [(8, 200, 300, 400, 500)[i % 5] for i in range(26)]          # too many sizes for a launch each


@pytest.mark.parametrize("dims,sizes,periodic,alg,want", [
    ((32, 32, 32), FIVE, None, 0, True), ((32, 32, 32), FIVE, None, 1, True), ((32, 32, 32), FIVE, None, 5, False), ((32, 32, 32), FIVE, (0, 0, 0), 0, False),
    ((20, 20, 20), FIVE, None, 0, False), ((32, 32, 32), [max(200, x) for x in FIVE], None, 0, False), ((32, 32, 32), 64, None, 5, False), ((32, 32, 32), 64, (0, 0, 0), 0, False),
    ((24, 24, 24), 25, None, 0, False), ((64, 64, 64), 11, None, 0, False)])
def test_small_and_large_blocks_by_their_size(stub_library, dims, sizes, periodic, alg, want):
    """Blocks of up to 128 bytes and larger ones in one launch, a quarter of the cache and more; 11 x 11 is not larger."""
    sizes = sizes if isinstance(sizes, list) else [int(x) for x in gen.stencil_block_sizes(gen.moore(3, 1), sizes)]
    got = _policies(stub_library.start_unequal(dims, gen.moore(3, 1), alg, sizes, periodic))
    assert (("block", 4) in got) == want, got


@pytest.mark.parametrize("dims,offsets,m,layout,push", [
    ((50, 50, 50), gen.von_neumann(3, 1), 64, 0, 0), ((32, 32, 32), gen.von_neumann(3, 1), 1056, 0, 0),
    ((50, 50, 50), gen.von_neumann(3, 1), 128, 0, 3), ((50, 50, 50), gen.von_neumann(3, 1), 1024, 0, 3),
    ((50, 50, 50), gen.von_neumann(3, 1), 100, 1, 3), ((32, 32, 32), gen.moore(3, 1), 192, 0, 2),
    ((32, 32, 32), gen.moore(3, 1), 256, 0, 3), ((32, 32, 32), gen.moore(3, 1), 200, 0, 0)])
def test_allgather_rounds_that_read_a_block_once(stub_library, dims, offsets, m, layout, push):
    """How many of the three launches take the push form: two moves from one block only as whole lines or dense planes."""
    got = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_COMBINED_BYDIM, m, layout))
    assert len(got) == 3 and got.count("shift_push_kernel") == push


@pytest.mark.parametrize("dims,offsets,m,eighths", [((250000,), gen.von_neumann(1, 1), 256, False), ((60, 50, 41), gen.moore(3, 1), 200, True),
                                                    ((250, 250), gen.von_neumann(2, 1), 256, True), ((4099,), gen.von_neumann(1, 2), 8192, True)])
def test_fused_allgather_takes_eighths_where_a_run_does_not_hold_the_neighbourhood(stub_library, dims, offsets, m, eighths):
    got = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_SX_FUSED, m))
    assert got == ["vector_round_kernel"] or got == ["vector_round_uniform_kernel"]
    tiles = -(-int(np.prod(dims)) * len(offsets) * (-(-m // 16)) // 256)
    assert tiles % 1024 and stub_library.grids == [-(-tiles // 8) * 8 if eighths else -(-tiles // 1024) * 1024]


def test_interior_tiles_of_mesh_launches(tmp_path):
    import stub_library as sl
    exe = sl.build_driver(str(tmp_path), "mesh_tiles_driver.cpp")
    proc = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert proc.returncode == 0 and "mesh tiles ok" in proc.stdout, proc.stdout


def test_interior_units_and_packed_coordinates_of_mesh_launches(tmp_path):
    import stub_library as sl
    exe = sl.build_driver(str(tmp_path), "mesh_units_driver.cpp")
    proc = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert proc.returncode == 0 and "mesh units ok" in proc.stdout, (proc.returncode, proc.stdout)


@pytest.mark.parametrize("alg", [iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM])
def test_binding_a_large_box_is_no_walk_over_its_tiles(stub_library, alg):
    """Init binds two launch lists (rounds one by one, and as iso_start takes them): one copy to the device for both,
    and milliseconds less than a walk over the tiles of a 64^3 box takes (22 ms for both lists; here 0.4)."""
    dims, offsets, m = (64, 64, 64), gen.moore(3, 1), 200
    p, s, niso = 64 ** 3, len(offsets), stub_library.iso
    comm = stub_library.comm(dims, offsets, (0, 0, 0))
    with stub_library.buffers(p * s * m, p * s * m, niso.iso_workspace_bytes(comm, 0, alg, m)) as bufs:
        best = 1.0
        for _ in range(5):
            copies, t0 = stub_library.lib.stub_copies(), time.perf_counter()
            req = stub_library.request(comm, dims, s, 0, alg, m, 0, bufs)
            best = min(best, time.perf_counter() - t0)
            assert stub_library.lib.stub_copies() == copies + 1
            niso.iso_request_free(req)
    assert best < 4e-3, best


def test_merged_rounds_of_many_entries_bind_in_little_more_time(stub_library):
    """16 806 neighbours: init that also merges the rounds of a dimension, against one whose plan has one round per
    dimension from the start (1.1 times its time; 1.5 to 1.8 times under a comparison sort of the entries and a table
    that grows and is copied).  As many tries as it takes to see the shortest of both."""
    dims, offsets, m = (5, 4, 4, 3, 2), gen.moore(5, 3), 8
    p, s = int(np.prod(dims)), len(offsets)
    comm = stub_library.comm(dims, offsets)
    algs = iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM
    need = max(stub_library.iso.iso_workspace_bytes(comm, iso.ISO_OP_ALLTOALL, alg, m) for alg in algs)
    best = {alg: 1.0 for alg in algs}
    with stub_library.buffers(p * s * m, p * s * m, need) as bufs:
        for _ in range(60):
            for alg in algs:
                t0 = time.perf_counter()
                req = stub_library.request(comm, dims, s, iso.ISO_OP_ALLTOALL, alg, m, iso.ISO_LAYOUT_RANK_MAJOR, bufs)
                best[alg] = min(best[alg], time.perf_counter() - t0)
                stub_library.iso.iso_request_free(req)
            if best[algs[0]] < 1.3 * best[algs[1]]:
                break
    assert best[algs[0]] < 1.3 * best[algs[1]], best


@pytest.mark.parametrize("dims,offsets,m,layout,op,kernels", [
    ((16, 16, 16, 16), gen.random_distinct(4, -3, 3, 40, 5), 1024, 0, 0, 24), ((32, 32, 32), gen.random_distinct(3, -3, 3, 40, 5), 1024, 0, 0, 18),
    ((8,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 1024, 1, 0, 5), ((16,) * 4, gen.random_distinct(4, -3, 3, 40, 5), 256, 1, 0, 4),
    ((32, 32, 32), gen.random_distinct(3, -3, 3, 40, 5), 1024, 1, 0, 3), ((9,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 512, 0, 0, 30), ((48, 48, 48), gen.moore(3, 2), 128, 0, 0, 12),
    ((8,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 256, 0, 0, 5), ((10,) * 4, gen.random_distinct(4, -3, 3, 40, 5), 400, 0, 0, 4),
    ((64, 64, 64), gen.moore(3, 1), 128, 0, 0, 3), ((128, 128), gen.moore(2, 3), 2048, 0, 0, 2),
    ((48, 48, 48), gen.moore(3, 2), 128, 0, 1, 3), ((8, 8), gen.moore(2, 1), 32, 0, 0, 2)])
def test_mesh_rounds_go_together_where_that_does_not_cost_their_interior(stub_library, dims, offsets, m, layout, op, kernels):
    names = _names(stub_library.start(dims, offsets, op, iso.ISO_ALG_COMBINED, m, layout, (0,) * len(dims)))
    assert names == kernels * ["mesh_shift_round_kernel"]


@pytest.mark.parametrize("op", [iso.ISO_OP_ALLTOALL, iso.ISO_OP_ALLGATHER])
@pytest.mark.parametrize("alg", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("dims,offsets,m", [((8, 8), gen.moore(2, 1), 32), ((32, 32, 32), gen.moore(3, 1), 256), ((12, 13), gen.von_neumann(2, 2), 4000)])
def test_start_info_says_what_a_start_enqueues(stub_library, dims, offsets, m, alg, op):
    """The number of kernels, and the bytes of the blocks that they load and store: every move stores one; an allgather's
    moves out of one block load it once per kernel; one kernel for all hops loads the send buffer, and the one for the
    staged schedule's first two rounds every block of a row that makes a hop in them."""
    niso, p, s = stub_library.iso, int(np.prod(dims)), len(offsets)
    comm = stub_library.comm(dims, offsets)
    with stub_library.buffers(p * m * s, p * s * m, niso.iso_workspace_bytes(comm, op, alg, m)) as bufs:
        req = stub_library.request(comm, dims, s, op, alg, m, 0, bufs)
        info, plan = niso.iso_request_info(req), niso.iso_request_plan(req)
        rounds = [niso.iso_plan_entries(plan, q) for q in range(niso.iso_plan_info(plan)["launches"])]
        moves = [e for r in rounds for e in r]
        for graph in (niso.ISO_GRAPH_OFF, niso.ISO_GRAPH_CHAIN):
            niso.iso_request_set_graph(req, graph)
            got = niso.iso_request_start_info(req)
            if graph:
                assert got["kernels"] == info["launches"]
            else:
                assert got["kernels"] == len(stub_library.launched(lambda: niso.iso_start(req, 0)))
            joined = got["kernels"] < len([r for r in rounds if r]) and alg == 5 and op == iso.ISO_OP_ALLTOALL and len(dims) == 3
            if got["kernels"] == 1:
                assert got["bytes_read"] == p * m * (s if op == iso.ISO_OP_ALLTOALL else 1)
            elif joined and not graph:
                early = {e["neighbor"] for r in rounds[:2] for e in r}
                assert len(early) == 20 and got["bytes_read"] == (len(early) + s) * p * m
            elif op == iso.ISO_OP_ALLTOALL:
                assert got["bytes_read"] == info["bytes_read"]
            else:
                sources = len({(e["src_buf"], e["src_slot"]) for e in moves})
                assert sources * p * m <= got["bytes_read"] <= info["bytes_read"]
            assert got["bytes_written"] == info["bytes_written"]
        niso.iso_request_free(req)


A2A, LINES, TAIL = "vector_round_kernel<v16, 3, true, 0, false, 1>", "vector_round_kernel<v16, 3, true, 1, false, 1>", "vector_round_kernel<v16, 3, true, 0, true, 1>"


@pytest.mark.parametrize("dims,offsets,m,layout,alg,kernel", [
    ((9, 9, 9), gen.moore(3, 1), 256, 0, 0, A2A), ((8, 8, 8), gen.moore(3, 1), 256, 0, 0, None), ((9, 9, 9), gen.moore(3, 1), 256, 0, 1, A2A),
    ((20, 20, 20), gen.moore(3, 1), 128, 0, 0, A2A), ((17, 17, 17), gen.moore(3, 1), 128, 0, 0, None), ((22, 22, 22), gen.moore(3, 1), 128, 0, 1, A2A), ((20, 20, 20), gen.moore(3, 1), 128, 0, 1, None),
    ((32, 32, 32), gen.moore(3, 1), 1027, 0, 0, TAIL), ((12, 12, 12), gen.moore(3, 1), 600, 0, 1, None), ((12, 12, 12), gen.moore(3, 1), 600, 0, 0, TAIL),
    ((32, 32, 32), gen.moore(3, 1), 319, 0, 0, None), ((32, 32, 32), gen.moore(3, 1), 320, 0, 0, A2A), ((12, 12, 12), gen.moore(3, 1), 400, 0, 0, None),
    ((32, 32, 32), gen.moore(3, 1), 400, 0, 1, None), ((40, 40, 40), gen.moore(3, 1), 320, 0, 1, A2A), ((64, 64, 64), gen.moore(3, 1), 256, 0, 1, LINES),
    ((32, 32, 32), gen.moore(3, 1), 1024, 0, 0, "vector_round_uniform_kernel<3, 1, 1>"), ((32, 32, 32), gen.moore(3, 1), 100, 1, 0, TAIL), ((20, 20, 20), gen.moore(3, 1), 128, 1, 0, None),
    ((16, 16, 16, 16), gen.random_distinct(4, -3, 3, 30, 5), 128, 0, 0, "vector_round_kernel<v16, 5, true, 1, false, 1>"),
    ((20, 20, 20), gen.moore(3, 2), 320, 0, 0, A2A), ((20, 20, 20), gen.moore(3, 2) + [(3, 3, 3)] * 5, 320, 0, 0, A2A + " " + A2A),
    ((3, 3, 3, 3, 3, 3), gen.moore(6, 1)[:100], 1024, 0, 0, None)])
def test_alltoalls_through_all_hops_in_one_launch(stub_library, dims, offsets, m, layout, alg, kernel):
    """Whole lines (from 256 bytes on) from 4 MiB on, others by block and size; up to five dimensions, a launch for every 128 neighbours."""
    got = stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m, layout)
    assert " ".join(got) == kernel if kernel else len(got) > 1 or got[0].startswith("chain"), got
    assert len(stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, alg, m, layout, by_rounds=True)) > 1


PULL, PULL_TAIL = "vector_round_kernel<v16, 3, true, 0, false, 0>", "vector_round_kernel<v16, 3, true, 0, true, 0>"


@pytest.mark.parametrize("dims,offsets,m,layout,alg,kernel", [
    ((12, 12, 12), gen.moore(3, 1), 128, 0, 0, PULL), ((10, 10, 10), gen.moore(3, 1), 128, 0, 0, None),
    ((20, 20, 20), gen.moore(3, 1), 256, 0, 1, PULL), ((33, 33, 33), gen.moore(3, 1), 256, 0, 1, None), ((33, 33, 33), gen.moore(3, 1), 256, 0, 0, PULL),
    ((33, 33, 33), gen.moore(3, 1), 512, 0, 1, PULL), ((64, 64, 64), gen.moore(3, 1), 128, 0, 1, PULL), ((28, 28, 28), gen.moore(3, 1), 255, 0, 0, None),
    ((20, 20, 20), gen.moore(3, 1), 255, 0, 0, PULL_TAIL), ((20, 20, 20), gen.moore(3, 1), 40, 0, 0, PULL_TAIL), ((37, 37, 37), gen.moore(3, 1), 40, 0, 0, None),
    ((40, 40, 40), gen.moore(3, 1), 40, 1, 0, PULL_TAIL), ((40, 40, 40), gen.random_distinct(3, -3, 3, 20, 5), 300, 0, 0, "vector_round_kernel<v16, 3, true, 0, true, 2>"),
    ((40, 40, 40), gen.random_distinct(3, -3, 3, 20, 5), 1024, 0, 0, "vector_round_uniform_kernel<3, 0, 2>"),
    ((8,) * 5, gen.random_distinct(5, -3, 3, 30, 5), 1024, 0, 0, "push_round_kernel<v16, 5, false, 2>"),
    ((8,) * 5, gen.random_distinct(5, -3, 3, 30, 5), 500, 0, 0, "vector_round_kernel<v16, 5, true, 0, true, 2>"),
    ((8,) * 5, gen.random_distinct(5, -3, 3, 30, 5), 500, 1, 0, "push_round_kernel<v16, 5, true, 0>"),
    ((8,) * 5, gen.random_distinct(5, -3, 3, 40, 5), 1024, 0, 0, "push_round_kernel<v16, 5, false, 2> push_round_kernel<v16, 5, false, 0>"),
    ((3,) * 6, gen.moore(6, 1)[:100], 1024, 0, 0, None)])
def test_allgathers_through_all_hops_in_one_launch(stub_library, dims, offsets, m, layout, alg, kernel):
    """From 4 MiB on, small blocks up to a part of the last-level cache; a launch for every 128 nodes of the trie."""
    got = stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, alg, m, layout)
    assert " ".join(got) == kernel if kernel else len(got) > 1, got
    assert len(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, alg, m, layout, by_rounds=True)) > 1


@pytest.mark.parametrize("dims,op,m,layout,alg,kernel", [
    ((45, 37, 29), 0, 100, 1, 1, "vector_round_kernel<v16, 3, true, 0, true, 5>"), ((45, 37, 29), 0, 100, 1, 0, None), ((45, 37, 29), 0, 100, 0, 1, None),
    ((45, 37, 29), 0, 256, 0, 1, "vector_round_kernel<v16, 3, true, 1, false, 5>"), ((45, 37, 29), 1, 256, 1, 1, "vector_round_kernel<v16, 3, true, 0, false, 4>"),
    ((45, 37, 29), 1, 600, 0, 1, "vector_round_kernel<v16, 3, true, 0, true, 4>"), ((45, 37, 29), 1, 300, 0, 1, None), ((45, 37, 29), 0, 1024, 0, 3, "vector_round_uniform_kernel<3, 1, 4>"),
    ((45, 37, 29), 1, 7, 0, 3, "vector_round_kernel<unsigned int, 3, true, 0, true, 4>"), ((45, 37, 29), 1, 1024, 1, 3, "vector_round_uniform_kernel<3, 0, 4>"),
    ((3, 4, 3, 4, 3, 4), 0, 64, 0, 3, "block_round_kernel<true, true, 0, false, 0>")])
def test_boxes_by_full_vectors(stub_library, dims, op, m, layout, alg, kernel):
    got = stub_library.start(dims, gen.moore(3, 1) if len(dims) == 3 else gen.von_neumann(6, 1), op, alg, m, layout, (0,) * len(dims))
    assert got == [kernel] if kernel else len(got) > 1, got


@pytest.mark.parametrize("dims,sizes,alg,kernels", [
    ((32, 32, 32), gen.stencil_block_sizes(gen.moore(3, 1), 64), 0, "vector_round_uniform_kernel<3, 1, 1> block_round_kernel<true, true, 2, false, 3>"),
    ((32, 32, 32), gen.stencil_block_sizes(gen.moore(3, 1), 25), 1, "vector_round_kernel<v16, 3, true, 0, true, 1> block_round_kernel<true, true, 2, false, 3>"),
    ((32, 32, 32), gen.stencil_block_sizes(gen.moore(3, 1), 64), 1, "vector_round_uniform_kernel<3, 1, 1> block_round_kernel<true, true, 2, false, 3>"), ((64, 64, 64), gen.stencil_block_sizes(gen.moore(3, 1), 12), 0, "vector_round_kernel<v16, 3, true, 0, false, 1> block_round_kernel<true, true, 2, false, 3>"),
    ((32, 32, 32), gen.stencil_block_sizes(gen.moore(3, 1), 25), 0, "vector_round_kernel<v16, 3, true, 0, true, 1> block_round_kernel<true, true, 2, false, 3>"),
    ((20, 20, 20), gen.stencil_block_sizes(gen.moore(3, 1), 25), 0, "vector_round_kernel<v16, 3, true, 0, true, 1> block_round_kernel<true, true, 2, false, 3>"),
    ((20, 20, 20), gen.stencil_block_sizes(gen.moore(3, 1), 8), 0, "block_round_kernel<true, true, 2, false, 3>"), ((20, 20, 20), gen.stencil_block_sizes(gen.moore(3, 1), 8), 1, None),
    ((20, 20, 20), gen.stencil_block_sizes(gen.moore(3, 1), 9), 0, None),
    ((8, 8, 8), [200 + 16 * (i % 2) for i in range(26)], 0, "vector_round_kernel<v16, 3, true, 0, true, 1> vector_round_kernel<v16, 3, true, 0, true, 1>"),
    ((8, 8, 8), [200 + 16 * (i % 2) for i in range(25)] + [8], 0, None)])
def test_unequal_blocks_by_size(stub_library, dims, sizes, alg, kernels):
    """Fewer launches than dimensions: one for every size of more than eight units, one for all smaller blocks."""
    got = stub_library.start_unequal(dims, gen.moore(3, 1), alg, list(sizes))
    assert " ".join(got) == kernels if kernels else all(k.startswith("block_round_kernel<true, false, ") and k.endswith(", 0>") for k in got), got


@pytest.mark.parametrize("dims,offsets,m,kernels", [
    ((64, 64, 64), gen.moore(3, 1), 16, "staged_round_kernel<v16, 2, 4u, false, true> deliver_kernel<v16, 0, 4u>"),
    ((40, 40, 40), gen.moore(3, 1), 64, "staged_round_kernel<v16, 0, 4u, false, true> deliver_kernel<v16, 0, 4u>"),
    ((32, 32, 32), gen.moore(3, 2), 256, "staged_round_kernel<v16, 1, 8u, false, true> deliver_kernel<v16, 1, 8u>"),
    ((100, 100), gen.moore(2, 1), 64, None), ((20, 20, 20), gen.moore(3, 1), 40, None)])
def test_first_two_rounds_of_the_staged_schedule(stub_library, dims, offsets, m, kernels):
    """One launch for both where the rounds are re-tiled: whole units, or beyond 48 MiB."""
    got = stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, m)
    assert " ".join(got) == kernels if kernels else not any(k.endswith("true>") for k in got), got


@pytest.mark.parametrize("dims,offsets,sizes,kernels", [
    ((32, 32), gen.moore(2, 10), [4 + 4 * (i % 2) for i in range(440)], 2), ((32, 32), gen.moore(2, 5), [4 + 4 * (i % 2) for i in range(120)], 1),
    ((8, 8, 8), gen.moore(3, 3), [4 + 4 * (i % 2) for i in range(342)], 3), ((8, 8, 8), gen.moore(3, 3)[:256], [4 + 4 * (i % 2) for i in range(256)], 2),
    ((8,) * 5, [(i, 0, 0, 0, 0) for i in (1, 2, 3, 4)], [200, 300, 400, 500], 1), ((8,) * 5, [(i, 0, 0, 0, 0) for i in (1, 2, 3, 4)], [20, 30, 40, 50], 1),
    ((8,) * 4, [(1, 0, 0, 0), (2, 0, 0, 0), (0, 3, 0, 0), (0, 2, 0, 0), (1, 1, 0, 0)], [200, 300, 400, 200, 300], 2)])
@pytest.mark.parametrize("box", [False, True])
def test_unequal_blocks_take_no_more_launches_than_one_per_dimension(stub_library, dims, offsets, sizes, kernels, box):
    """Launches and not sizes count, each of at most 128 blocks, against the dimensions that some block moves along."""
    offsets = [tuple(int(x) for x in c) for c in offsets]
    got = stub_library.start_unequal(dims, offsets, iso.ISO_ALG_COMBINED, sizes, (0,) * len(dims) if box else None)
    assert len(got) == kernels, got


@pytest.mark.parametrize("dims,offsets,m,op,kernels", [
    ((5, 5), gen.moore(2, 10), 384, 0, ["chain_kernel"]), ((5, 5), gen.moore(2, 10), 768, 1, ["chain_kernel"]), ((7, 7), gen.moore(2, 7), 768, 0, ["chain_kernel"]),
    ((5, 5), gen.moore(2, 10), 4480, 0, 3), ((5, 5), gen.moore(2, 10), 4480, 1, 3), ((8, 8), gen.moore(2, 15), 768, 1, 3), ((3, 3, 3), gen.moore(3, 4), 1280, 0, 4),
    ((8, 8), gen.moore(2, 15), 6784, 0, ["vector_round_kernel"] * 8), ((32, 32), gen.moore(2, 10), 384, 0, ["vector_round_kernel"] * 4), ((32, 32), gen.moore(2, 10), 256, 0, 2), ((5, 5, 5), gen.moore(3, 3), 384, 0, ["vector_round_kernel"] * 3)])
@pytest.mark.parametrize("alg", [iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM])
def test_more_neighbours_than_one_table_takes(stub_library, dims, offsets, m, op, kernels, alg):
    """The chain stays, and up to 32 MiB a launch and the size of the last-level cache so do fewer launches."""
    got = _names(stub_library.start(dims, offsets, op, alg, m))
    assert got == kernels if isinstance(kernels, list) else len(got) == kernels and "vector_round_kernel" not in got, got


@pytest.mark.parametrize("dims,n,m,policy", [
    ((9, 8, 8, 9, 8), 40, 16, 2), ((16, 16, 15, 15), 30, 20, 2), ((7,) * 5, 40, 56, 2), ((7,) * 5, 40, 64, 0), ((12, 12, 11, 12, 12), 10, 20, 2),
    ((12, 12, 11, 12, 12), 10, 16, 0), ((16, 16, 16, 15), 10, 32, 0), ((24, 25, 24), 40, 16, 0), ((40, 40, 36), 40, 20, 0)])
def test_small_allgather_blocks_through_all_hops_meet_in_the_caches(stub_library, dims, n, m, policy):
    """More than 32 trie nodes beside the receive blocks, or more than half the cache to write: plain stores under a sector."""
    offsets = gen.random_distinct(len(dims), -3, 3, n, gen.configs.CONFIG5_NEIGHBOURHOOD_SEED)
    for alg in (iso.ISO_ALG_COMBINED, iso.ISO_ALG_COMBINED_BYDIM):
        (got,) = stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, alg, m)
        assert got.endswith(", 2>") and _policies([got]) == {("vector", policy)}, got


@pytest.mark.parametrize("dims,offsets,m,push", [
    ((191, 177), gen.moore(2, 2), 640, True), ((41, 49, 53), gen.von_neumann(3, 2), 192, True), ((12, 10, 10, 10), gen.von_neumann(4, 2), 1813, True),
    ((20, 20, 20), gen.moore(3, 1), 992, True), ((20, 20, 20), gen.moore(3, 1), 1024, False), ((20, 20, 20), gen.moore(3, 1), 1040, False), ((20, 20, 20), gen.moore(3, 1), 1072, False),
    ((20, 20, 20), gen.moore(3, 1), 1088, True), ((20, 20, 20), gen.moore(3, 1), 1304, False), ((20, 20, 20), gen.moore(3, 1), 1320, True), ((20, 20, 20), gen.moore(3, 1), 1296, True),
    ((20, 20, 20), gen.moore(3, 1), 784, False), ((64, 64, 64), gen.moore(3, 1), 32, False), ((64, 64, 64), gen.moore(3, 1), 128, True), ((45, 37, 29), gen.moore(3, 1), 128, False)])
def test_slot_major_allgathers_through_all_hops_where_planes_do_not_meet(stub_library, dims, offsets, m, push):
    """From 6 MiB to send on: pushed, unless a plane is a multiple of the runs of all XCDs, or of half of them; above 28 MiB always."""
    (got,) = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_COMBINED, m, iso.ISO_LAYOUT_SLOT_MAJOR))
    assert (got == "push_round_kernel") == push, got


@pytest.mark.parametrize("dims,offsets,m,want", [
    ((250, 260), gen.moore(2, 1), 5600, 2), ((250, 260), gen.von_neumann(2, 2), 4416, 2), ((250, 260), gen.random_distinct(2, -3, 3, 10, 5), 6432, 2), ((250, 260), gen.moore(2, 1), 4240, "vector_round_kernel"), ((250, 260), gen.moore(2, 1), 5601, "vector_round_kernel"),
    ((250, 260), gen.moore(2, 1), 5120, "push_round_kernel"), ((400, 420), gen.moore(2, 1), 2048, "push_round_kernel"), ((250, 260), gen.moore(2, 1), 4096, "vector_round_uniform_kernel"),
    ((64, 64, 64), gen.moore(3, 1), 1168, "vector_round_kernel")])
def test_allgathers_of_more_than_the_cache_holds(stub_library, dims, offsets, m, want):
    """Whole lines are pushed; other whole units stay a launch per dimension in two dimensions."""
    got = _names(stub_library.start(dims, offsets, iso.ISO_OP_ALLGATHER, iso.ISO_ALG_COMBINED, m))
    assert got == [want] if isinstance(want, str) else len(got) == want and got[0].startswith("shift"), got


@pytest.mark.parametrize("dims,edge,box,joined", [
    ((64, 64, 64), 3, False, False), ((64, 64, 64), 2, False, False), ((64, 64, 64), 4, False, True), ((32, 32, 32), 3, False, True), ((48, 48, 48), 3, False, False),
    ((512, 512), 3, False, False), ((512, 512), 11, False, False), ((512, 512), 15, False, True), ((200, 200), 3, False, True), ((512, 512), 3, True, True),
    ((360, 360), 3, False, False), ((360, 360), 4, False, True), ((400, 400), 4, False, True), ((450, 450), 4, False, False),
    ((16,) * 4, 2, False, False), ((9,) * 5, 2, False, False), ((8,) * 5, 4, False, True), ((64, 64, 64), 8, True, False), ((64, 64, 64), 8, False, True), ((64, 64, 64), 4, True, False),
    ((32, 32, 32), 8, True, True), ((64, 64, 64), 16, True, True), ((20,) * 4, 4, True, False)])
def test_blocks_of_a_few_bytes_on_large_tori(stub_library, dims, edge, box, joined):
    """A launch per dimension for blocks of a few bytes, and on boxes for small ones alone, from a million units or more on."""
    sizes = [int(x) for x in gen.stencil_block_sizes(gen.moore(len(dims), 1), edge)]
    got = stub_library.start_unequal(dims, gen.moore(len(dims), 1), iso.ISO_ALG_COMBINED, sizes, (0,) * len(dims) if box else None)
    assert (len(got) < len(dims)) == joined, got


@pytest.mark.parametrize("dims,n,m,units", [((8,) * 5, 40, 208, 8), ((8,) * 5, 40, 224, 8), ((8,) * 5, 40, 112, 8), ((8,) * 5, 40, 192, 4), ((8,) * 5, 40, 160, 4),
                                            ((5,) * 5, 40, 208, 4), ((8,) * 5, 40, 107, 8), ((8,) * 5, 40, 90, 4)])
def test_tiles_of_the_first_two_staged_rounds(stub_library, dims, n, m, units):
    """Large ones where few ranks of a small tile end inside a sector, beyond half the last-level cache."""
    offsets = gen.random_distinct(5, -3, 3, n, gen.configs.CONFIG5_NEIGHBOURHOOD_SEED)
    got = stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, m)
    assert got[0].startswith("staged_round_kernel") and got[0].endswith("true>") and f", {units}u, " in got[0], got


@pytest.mark.parametrize("dims,offsets,m,two", [
    ((32, 32, 32), gen.von_neumann(3, 2), 256, True), ((48, 48, 48), gen.von_neumann(3, 2), 240, False), ((48, 48, 48), gen.moore(3, 1), 240, True),
    ((18,) * 4, gen.von_neumann(4, 2), 160, False), ((13,) * 4, gen.von_neumann(4, 2), 160, True)])
def test_first_two_staged_rounds_that_share_no_block(stub_library, dims, offsets, m, two):
    """In one launch up to the size of the last-level cache."""
    got = stub_library.start(dims, offsets, iso.ISO_OP_ALLTOALL, iso.ISO_ALG_COMBINED_STAGED, m)
    assert any(k.startswith("staged_round_kernel") and k.endswith("true>") for k in got) == two, got
