"""The launch rules (which kernel shape a call takes), evaluated on the host: each case names the side of
a rule that a GPU test or a measurement stands on, so that a changed rule cannot move it silently."""
import ctypes

import pytest

import paper_2606_07684_amd as scd

DECODE, PATCH, ENCODE_KV = 0, 1, 2
K128X64, K128X32, K32X64, K32X32, STAGED = range(5)


class _Job(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("a", "b", "c", "vec")] + [
        (n, ctypes.c_int32) for n in ("n", "k", "flags", "tile_begin")]


def _rule(symbol, res, *args):
    fn = getattr(scd.load_library(), symbol)
    fn.restype, fn.argtypes = res, list(args)
    return fn


def generic_shape(op, bf16, m, jobs):
    arr = (_Job * len(jobs))(*[_Job(None, None, None, None, n, k, 0, 0) for n, k in jobs])
    fn = _rule("_ZN3scd13generic_shapeENS_2OpEbPKNS_7GemmJobEml", ctypes.c_int, ctypes.c_int,
               ctypes.c_bool, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int64)
    return fn(op, bf16, arr, len(jobs), m)


@pytest.mark.parametrize("op,bf16,tokens,jobs,want", [
    # bf16 decode: more than 256 requests of an 8-head model, heads of 32, a short prefix, heads' shared rows
    (DECODE, True, 32768, [(1024, 128)] * 56, STAGED), (DECODE, True, 8192, [(512, 64)] * 16, STAGED),
    (DECODE, True, 64, [(512, 64)] * 16, K128X32), (DECODE, True, 131072, [(64, 64)] * 8, K128X64),
    (DECODE, True, 262144, [(32, 32)] * 12, K128X32),
    # bf16 Patch: heads of 32, and a prefix whose contraction is better split
    (PATCH, True, 8192, [(512, 2048)] * 8, STAGED), (PATCH, True, 200, [(1024, 4128)] * 8, K32X64),
    # fp32 decode takes 16-byte stores of 32 x 64 waves; the key and value encode, by the last round
    (DECODE, False, 8192, [(1024, 128)] * 32, K128X64), (DECODE, False, 100, [(256, 32)] * 6, K128X32),
    (ENCODE_KV, False, 4099, [(64, 512)] * 16, K32X64), (ENCODE_KV, False, 8192, [(64, 512)] * 16, K128X64),
    (ENCODE_KV, False, 64, [(64, 512)] * 16, K32X32), (ENCODE_KV, True, 4099, [(128, 1024)] * 16, K128X64)])
def test_generic_shape(op, bf16, tokens, jobs, want):
    assert generic_shape(op, bf16, tokens, jobs) == want


# (rank, tokens, layers): the cases of test_gpu_tiles at w = 1024, and 28 layers of an 8-head model
@pytest.mark.parametrize("rank,tokens,layers,want", [
    (128, 40, 2, 1), (128, 1999, 7, 2), (128, 8192, 4, 4), (256, 333, 2, 1), (256, 5000, 2, 2), (64, 500, 3, 1),
    (64, 31000, 2, 2), (64, 40000, 2, 4), (32, 9000, 4, 2), (32, 31000, 2, 4), (32, 40000, 2, 4),
    (16, 65700, 1, 4), (48, 65700, 1, 4), (112, 65700, 1, 4), (128, 1100, 48, 4), (256, 1100, 24, 2),
    (32, 1000, 28, 4), (48, 2000, 28, 4), (64, 2000, 28, 2), (32, 333, 28, 2), (128, 2000, 28, 4), (256, 700, 28, 2)])
def test_decode_chunks(rank, tokens, layers, want):
    fn = _rule("_ZN3scd21decode_channel_groupsEiill", ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int64,
               ctypes.c_int64)
    assert fn(rank, 1024, tokens, layers) == want


# (w, rank, rows, layers): the cases of test_gpu_tiles.test_encode_shapes, and both sides of each line
@pytest.mark.parametrize("w,rank,rows,layers,want", [
    (1024, 256, 303, 1, True), (1024, 128, 5000, 2, True), (256, 64, 9100, 8, False), (256, 96, 9001, 8, False),
    (512, 128, 700, 1, True), (512, 128, 40000, 2, True), (512, 96, 30100, 3, True), (256, 96, 33000, 4, True),
    (128, 32, 131080, 4, True), (128, 64, 131080, 4, True), (128, 128, 23992, 1, False),
    (128, 64, 800, 16, False), (128, 64, 65536, 28, True),
    (1024, 64, 1500, 14, True), (1024, 64, 2000, 14, False), (512, 64, 1000, 24, True), (512, 64, 4000, 24, False),
    (512, 96, 4000, 24, True), (256, 128, 4000, 24, False), (256, 128, 16384, 24, True),
    (1024, 128, 333, 24, True), (1024, 128, 8192, 28, False)])
def test_encode_resident(w, rank, rows, layers, want):
    fn = _rule("_ZN3scd15encode_residentEiill", ctypes.c_bool, ctypes.c_int, ctypes.c_int, ctypes.c_int64,
               ctypes.c_int64)
    assert fn(w, rank, rows, layers) == want


# Jobs per launch: a full table, and where its workgroups of 256 threads would be 2^32 work-items (64 jobs of
# 1024 columns in 128 x 32 tiles from 1,048,576 rows on), fewer; one job always fits.
@pytest.mark.parametrize("rows,n,jobs,bm,bn,want", [
    (8192, 1024, 70, 128, 32, 64), (8192, 1024, 5, 128, 64, 5), (1048448, 1024, 64, 128, 32, 64),
    (1048576, 1024, 64, 128, 32, 63), (8388608, 1024, 64, 128, 32, 7), (8388608, 1024, 64, 128, 128, 31),
    (2 ** 31 - 1, 32, 3, 128, 32, 1)])
def test_launch_jobs(rows, n, jobs, bm, bn, want):
    arr = (_Job * jobs)(*[_Job(None, None, None, None, n, 64, 0, 0) for _ in range(jobs)])
    fn = _rule("_ZN3scd11launch_jobsEPKNS_7GemmJobEmlii", ctypes.c_size_t, ctypes.c_void_p, ctypes.c_size_t,
               ctypes.c_int64, ctypes.c_int, ctypes.c_int)
    assert fn(arr, jobs, rows, bm, bn) == want


@pytest.mark.parametrize("launches,mib,want", [
    (2, 0, False), (2, 1, False), (3, 18, True), (3, 19, False), (6, 72, True), (6, 94, False)])
def test_decode_one_launch(launches, mib, want):
    fn = _rule("_ZN3scd17decode_one_launchEil", ctypes.c_bool, ctypes.c_int, ctypes.c_int64)
    assert fn(launches, mib << 20) == want
