"""bench.py's byte model of a PCG iteration against the arrays of the iteration's
kernels, counted one by one on a mesh of 2 x 2 x 2 hexahedra."""
import pytest

import bench


@pytest.mark.parametrize("s", [4, 8])
@pytest.mark.parametrize("N", [3, 4, 5, 7, 15])
def test_pcg_iteration_bytes(N, s):
    E, nodes = 8, (2 * N + 1) ** 3
    local, inner = E * (N + 1) ** 3, E * (N - 1) ** 3
    faced, shared = local - inner, nodes - inner  # local copies on element boundaries, and the nodes they are of
    own, halo = local, E * ((N + 3) ** 3 - (N + 1) ** 3)
    rec = E * 27 * 4 * 4
    factor = 1234
    arrays = [
        # operator: p, records, 8 vertices, A p at interiors, work array
        s * nodes, rec, s * E * 24, s * inner, s * faced,
        # r at the shared nodes: work array, r read and written
        s * faced, s * shared, s * shared,
        # r at the interiors and the restriction: records, r read, A p, r written, eight parts and their places
        rec, s * nodes, s * inner, s * inner, 8 * E * 8, 4 * E * 8,
        # coarse sweeps
        8 * factor,
        # patch solves: 125 + 26 records of two ints, or an int per patch node and outside slot; r; corrections
        *([8 * E * 125, 8 * E * 26] if N >= 5 else [4 * (own + halo), 4 * halo]), s * nodes, s * own, s * halo,
        # sum at the interiors: records, corrections, x and p read and written, work array
        rec, s * own, s * halo, 2 * s * inner, 2 * s * inner, s * faced,
        # at the shared nodes: work array, x and p read and written
        s * faced, 2 * s * shared, 2 * s * shared,
    ]
    assert bench.pcg_iteration_bytes(E, N, local, nodes, factor, s) == sum(arrays)


def test_patch_record_order_is_the_librarys():
    import os
    with open(os.path.join(os.path.dirname(bench.__file__), "paper_1506_05996_amd", "csrc", "sem_internal.h")) as f:
        assert f"kPatchRecordsFrom = {bench.PATCH_RECORDS_FROM};" in f.read()
