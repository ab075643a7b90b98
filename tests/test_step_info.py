"""Which kernels a GMRES step runs (psfd_step_info): host-side rules, no device."""
import ctypes as C

import pytest

INFINITY_CACHE = 256 << 20
ALWAYS = 2**31 - 1


def info(nx, ny, nz, step, precision=1):
    from paper_2606_25541_amd import _lib as L
    k = L.psfd_step_kernels()
    assert L.lib().psfd_step_info(nx, ny, nz, precision, step, C.byref(k)) == 0
    return k


@pytest.mark.parametrize("shape", [(64, 64, 32), (128, 128, 32), (128, 128, 64), (256, 256, 64), (64, 128, 8)])
def test_basis_is_read_past_the_caches_by_the_slots_in_use(shape):
    """Step j of a lock-step cycle works on slots 0 .. j + 1 and a workspace of their
    size: as many instances read them through the caches as fit, whatever the
    restart length, so an early step of a long cycle keeps its basis cached. A
    server's slots always do."""
    nx, ny, nz = shape
    slot = 3 * nx * ny * nz * 8
    for step in range(32):
        n = info(nx, ny, nz, step).cached_instances
        assert n * (step + 3) * slot <= INFINITY_CACHE < (n + 1) * (step + 3) * slot
    assert info(nx, ny, nz, -1).cached_instances == ALWAYS


def test_cached_steps_of_known_solves():
    # one 128 x 128 x 64 instance: every step of GMRES(8), the first steps of longer cycles
    assert [info(128, 128, 64, j).cached_instances >= 1 for j in (0, 7, 8, 29)] == [True, True, False, False]
    # ten 64 x 64 x 32 instances at restart 8: a basis of 283 MB, of which the first steps use little
    assert [info(64, 64, 32, j).cached_instances >= 10 for j in (0, 5, 6, 7)] == [True, True, False, False]
    # separate passes: not the kernels' choice
    assert info(32, 32, 32, 5).cached_instances == ALWAYS
    assert info(64, 64, 32, 5, precision=0).cached_instances == ALWAYS


@pytest.mark.parametrize("shape,want", [
    # (quarter planes, projections in the inverse kernel, update in the forward one, partials)
    ((64, 64, 32), (1, 1, 1, 384)), ((64, 64, 16), (1, 1, 0, 256)), ((64, 64, 8), (1, 1, 0, 256)),
    ((64, 64, 4), (0, 1, 0, 256)), ((128, 128, 64), (1, 1, 1, 768)), ((256, 64, 32), (1, 1, 1, 384)),
    ((256, 256, 64), (1, 1, 1, 768)), ((128, 128, 128), (1, 0, 0, 256)), ((32, 32, 32), (1, 0, 0, 256)),
    ((32, 16, 32), (0, 0, 0, 256))])
def test_gram_schmidt_kernels_by_shape(shape, want, monkeypatch):
    k = info(*shape, step=3)
    assert (k.quarter_planes, k.dots_in_inverse, k.update_in_forward, k.partials) == want
    # FP64 steps take the separate passes
    k = info(*shape, step=3, precision=0)
    assert (k.dots_in_inverse, k.update_in_forward, k.partials) == (0, 0, 512)
    # each switch takes its own work out; without the projections no fused update either
    monkeypatch.setenv("PSFD_FUSE_UPDATE", "0")
    assert info(*shape, step=3).update_in_forward == 0
    monkeypatch.delenv("PSFD_FUSE_UPDATE")
    monkeypatch.setenv("PSFD_FUSE_DOTS", "0")
    k = info(*shape, step=3)
    assert (k.dots_in_inverse, k.update_in_forward, k.partials) == (0, 0, 256)


@pytest.mark.parametrize("shape", [(64, 64, 32), (64, 64, 64), (64, 64, 8), (128, 128, 8), (128, 128, 16), (64, 64, 4),
                                   (32, 32, 32), (256, 64, 16), (128, 128, 128)])
def test_pending_givens_step_takes_no_launch(shape):
    """Square planes and quarter planes carry the Givens step of the column before in
    a kernel of the apply, in both precisions; row and column strips do not."""
    for precision in (0, 1):
        assert info(*shape, step=3, precision=precision).givens_launch == 0
    assert info(16, 8, 32, 3).givens_launch == 1


def test_fp64_square_planes_keep_one_block_per_plane():
    """FP64 steps of 64 x 64 planes: one block per plane at 32 and 64 z planes, quarter
    planes elsewhere and in FP32."""
    for nz in (8, 16, 32, 64, 128):
        assert info(64, 64, nz, 3, precision=0).quarter_planes == (nz not in (32, 64))
        assert info(64, 64, nz, 3).quarter_planes == 1
    assert info(64, 128, 32, 3, precision=0).quarter_planes == 1
    assert info(128, 128, 64, 3, precision=0).quarter_planes == 1


def test_step_info_rejects_bad_arguments():
    from paper_2606_25541_amd import _lib as L
    lib, k = L.lib(), L.psfd_step_kernels()
    assert lib.psfd_step_info(64, 64, 32, 1, 0, None) == L.PSFD_ERR_INVALID_ARG
    assert lib.psfd_step_info(64, 64, 32, 2, 0, C.byref(k)) == L.PSFD_ERR_INVALID_ARG
    assert lib.psfd_step_info(64, 64, 32, 1, -2, C.byref(k)) == L.PSFD_ERR_INVALID_ARG
    assert lib.psfd_step_info(48, 64, 32, 1, 0, C.byref(k)) == L.PSFD_ERR_UNSUPPORTED_SIZE


@pytest.mark.parametrize("shape,want", [((64, 64, 32), (True, True)), ((256, 64, 32), (True, True)),
                                        ((256, 256, 64), (True, True)), ((128, 128, 16), (True, False)),
                                        ((128, 128, 128), (False, False))])
def test_benchmark_counts_the_kernels_that_run(shape, want, monkeypatch):
    """bench.py counts the bytes of the step's kernels by the library's rules, on every
    grid and with the projections switched off."""
    import os
    import sys
    from types import SimpleNamespace
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import bench
    prob = SimpleNamespace(nx=shape[0], ny=shape[1], nz=shape[2])
    assert bench.gram_schmidt_in_transforms(prob) == want
    monkeypatch.setenv("PSFD_FUSE_DOTS", "0")
    assert bench.gram_schmidt_in_transforms(prob) == (False, False)
