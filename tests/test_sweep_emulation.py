"""The sweep kernels' own source, run on the CPU (no GPU needed).

tests/emu/hip/hip_runtime.h stands in for what the kernels use of HIP: lanes
are fibers that meet at barriers, ballots and DPP moves and take turns in
between in drawn orders; workgroups are threads.  What the compiler would be
told in inline assembly is taken out of a copy of csrc/, the rest is compiled
as it is.  So the strips and their two buffers, the halo and export plans, the
tickets and their order, the early sums, the chunk buffers, the line sweep's
ring and read-ahead and the packed sweep data are those that run on the GPU.

Checked for each sequence of sweeps: the sequential lexicographic sweep's bits
(the oracle's), no access outside an array (buffer accesses are checked, other
arrays end at a page that faults), no wait that times out, counters and buffer
word ready for the next launch, and sentinels in every entry of the strip
buffer that the next sweep uses.
"""
import concurrent.futures as cf
import ctypes as C
import hashlib
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import workloads

HERE = os.path.dirname(os.path.abspath(__file__))
EMU = os.path.join(HERE, "emu")
CSRC = os.path.join(os.path.dirname(HERE), "paper_2506_21932_amd", "csrc")
CLANG = next((c for c in ("/opt/rocm/lib/llvm/bin/clang++", shutil.which("amdclang++"), shutil.which("clang++"))
              if c and os.path.exists(c)), None)
SOURCES = ["smg_common.h", "smg_sweep.h", "smg_group.h", "smg_kernels.h", "wavefront.hip", "block.hip", "lgs.hip"]
LIBS = {"fp64": ("wavefront.hip", ["-DEMU_WAVEFRONT", "-DEMU_GROUP", "-DEMU_TYPE=double"]),
        "fp32": ("wavefront.hip", ["-DEMU_WAVEFRONT", "-DEMU_TYPE=float"]),
        "fp16": ("wavefront.hip", ["-DEMU_WAVEFRONT", "-DEMU_TYPE=__half"]),
        "block": ("block.hip", ["-DEMU_BLOCK"]),
        "line": ("lgs.hip", ["-DEMU_LINE"])}


def host_source(s):
    """The source without inline assembly, dynamic LDS from the emulation, and without the instantiations of the
    launchers (each library instantiates what it runs)."""
    s = re.sub(r'asm\("v_fma_mix_f32[^;]*op_sel:\[1[^;]*;', "r = emu::half_times(w, 1, sc);", s)
    s = re.sub(r'asm\("v_fma_mix_f32[^;]*;', "r = emu::half_times(w, 0, sc);", s)
    s = re.sub(r'asm(\s+volatile)?\(""[^;]*;', ";", s)
    s = re.sub(r"extern __shared__[^;]*\bunsigned char (\w+)\[\];", r"unsigned char* const \1 = EMU_DYN_LDS;", s)
    s = re.sub(r"\ntemplate hipError_t launch_[^;]*;", "", s)
    assert "asm" not in re.sub(r"//[^\n]*", "", s)
    return s


def build(tag):
    texts = {f: host_source(open(os.path.join(CSRC, f)).read()) for f in SOURCES}
    own = [open(os.path.join(EMU, f)).read() for f in ("sweeps.cpp", "hip/hip_runtime.h")]
    h = hashlib.sha256("".join(list(texts.values()) + own + LIBS[tag][1]).encode()).hexdigest()[:16]
    d = os.path.join(EMU, "_build", h)
    lib = os.path.join(d, tag + ".so")
    if not os.path.exists(lib):
        os.makedirs(d, exist_ok=True)
        src = os.path.join(d, f"src_{tag}_{os.getpid()}")
        os.makedirs(src, exist_ok=True)
        for f, t in texts.items():
            with open(os.path.join(src, f), "w") as fh:
                fh.write(t)
        tmp = lib + f".{os.getpid()}"
        subprocess.check_call([CLANG, "-x", "c++", "-std=c++17", "-O1", "-mfma", "-ffp-contract=off", "-w", "-fPIC",
                               "-shared", "-pthread", "-I" + EMU, "-I" + src, f'-DSMG_SOURCE="{LIBS[tag][0]}"',
                               *LIBS[tag][1], os.path.join(EMU, "sweeps.cpp"), "-o", tmp])
        os.replace(tmp, lib)
        shutil.rmtree(src)
    return lib


@pytest.fixture(scope="module")
def libs():
    if CLANG is None:
        pytest.skip("no clang++")
    with cf.ThreadPoolExecutor(len(LIBS)) as ex:
        return dict(zip(LIBS, (C.CDLL(p) for p in ex.map(build, LIBS))))


def ptr(a):
    return None if a is None else a.ctypes.data_as(C.c_void_p)


def ints(v):
    return (C.c_int * len(v))(*v)


FORWARD, BACKWARD = 1, -1
# grids of one tile and several (8 x 16 columns), ends inside, at and past a tile and a chunk of 16 steps, one point
# in an axis; directions in sequence, workgroups
SCALAR = [
    ((20, 35, 18), 27, 0, (1, -1), 3), ((20, 35, 18), 19, 0, (-1, 1), 2), ((20, 35, 18), 7, 0, (1, -1, -1), 2),
    ((20, 35, 18), 7, 1, (1, 1, -1), 3), ((9, 17, 40), 27, 0, (-1, -1, 1), 1), ((8, 16, 16), 27, 0, (1, -1), 1),
    ((7, 15, 33), 19, 0, (1, -1), 1), ((25, 8, 12), 27, 0, (1, -1), 0), ((25, 8, 12), 27, 1, (1, -1), 2),
    ((25, 8, 12), 19, 2, (-1, 1), 4), ((1, 50, 9), 19, 0, (1, -1), 2), ((40, 1, 5), 7, 0, (1, -1), 2),
    ((33, 33, 1), 27, 0, (1, -1), 4), ((12, 70, 3), 7, 0, (-1, 1), 3),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("shape,pat,tiles,dirs,cap", SCALAR, ids=lambda v: str(v))
def test_scalar(libs, shape, pat, tiles, dirs, cap, prec):
    g = workloads.rng(5)
    n = int(np.prod(shape))
    A = np.ascontiguousarray(workloads.random_sgdia(shape, pat, seed=3).reshape(pat, n))
    rd = 1.0 / A[pat // 2]
    npt = np.float64 if prec == "fp64" else np.float32
    h = g.uniform(-1, 1, size=(len(dirs),) + shape).astype(npt).astype(np.float64)
    a16 = sc = None
    Al = A.astype(npt)
    if prec == "fp16":
        sc = g.uniform(0.5, 2.0, size=n).astype(np.float32)
        half = A.astype(np.float16)
        a16, Al = half.view(np.uint16), sc * half.astype(np.float32)
    off = workloads.offsets(pat)
    for seed in (1, 2):
        x = np.empty_like(h)
        st = libs[prec].emu_scalar(ints(shape), pat, tiles, 0, len(dirs), ints(dirs), cap, C.c_ulong(seed), ptr(A),
                                   ptr(rd), ptr(a16), ptr(sc), ptr(h), ptr(x))
        assert st == 0
        for k, d in enumerate(dirs):
            ref = oracle.gs_sweep(off, Al, rd.astype(npt), h[k].astype(npt), np.zeros(shape, npt), d, 1)
            assert np.array_equal(x[k].astype(npt), ref), (seed, k)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("pat", [7, 19, 27])
def test_unit_diagonal(libs, pat, prec):
    shape, npt = (11, 20, 21), np.float64 if prec == "fp64" else np.float32
    A = np.ascontiguousarray(workloads.random_sgdia(shape, pat, seed=4).reshape(pat, -1)) / 32
    h = workloads.rng(6).uniform(-1, 1, size=shape).astype(npt).astype(np.float64)
    x, one = np.empty_like(h), np.ones(h.size)
    assert libs[prec].emu_scalar(ints(shape), pat, 0, 1, 1, ints([1]), 2, C.c_ulong(3), ptr(A), ptr(one), None, None,
                                 ptr(h), ptr(x)) == 0
    ref = oracle.gs_sweep(workloads.offsets(pat), A.astype(npt), one.astype(npt), h.astype(npt), np.zeros(shape, npt), 1, 1)
    assert np.array_equal(x.astype(npt), ref)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("dirn", [FORWARD, BACKWARD])
@pytest.mark.parametrize("pat", [7, 27])
def test_group(libs, pat, dirn, order):
    """Systems of a batch in one launch, few workgroups: one is not finite, one is finished (its output and strips
    stay as they are)."""
    dims = [(9, 17, 20), (8, 16, 12), (17, 18, 9), (5, 6, 7), (9, 17, 20)]
    bad, done = 1, 3
    As = [np.ascontiguousarray(workloads.random_sgdia(s, pat, seed=7 + k).reshape(pat, -1)) for k, s in enumerate(dims)]
    hs = [workloads.rng(8 + k).uniform(-1, 1, size=s) for k, s in enumerate(dims)]
    hs[bad][3, 3, 3] = np.nan
    A, h = (np.concatenate([v.ravel() for v in vs]) for vs in (As, hs))
    rd = np.concatenate([1 / a[pat // 2] for a in As])
    x = np.empty_like(h)
    live = [int(k != done) for k in range(len(dims))]
    for cap in (1, 3):
        assert libs["fp64"].emu_group(len(dims), ints(sum(dims, ())), pat, dirn, order, ints(live), cap, C.c_ulong(cap),
                                      ptr(A), ptr(rd), ptr(h), ptr(x)) == 0
        at = 0
        for k, s in enumerate(dims):
            got = x[at:at + hs[k].size].reshape(s)
            at += hs[k].size
            if k in (bad, done):
                assert not np.isfinite(got).all()
                continue
            ref = oracle.gs_sweep(workloads.offsets(pat), As[k], 1 / As[k][pat // 2], hs[k], np.zeros(s), dirn, 1)
            assert np.array_equal(got, ref), (cap, k)


@pytest.mark.parametrize("sh", [0, 1])
def test_tile_order(libs, sh):
    """Every tile once, and its producers -- (X-1, Y .. Y+sh), (X, Y-1) and (X-1, Y-1) -- before it."""
    for ntx in range(1, 20):
        for nty in range(1, 20):
            out = np.empty(ntx * nty, np.uint32)
            libs["fp64"].emu_tile_order(sh, ntx, nty, ptr(out))
            assert np.array_equal(np.sort(out), np.arange(ntx * nty))
            at = np.empty((ntx, nty), int)
            at[out // nty, out % nty] = np.arange(ntx * nty)
            assert (at[:, 1:] > at[:, :-1]).all() and (at[1:] > at[:-1]).all() and (at[1:, 1:] > at[:-1, :-1]).all()
            if sh:
                assert (at[1:, :-1] > at[:-1, 1:]).all()


# tiles of 4 x 8 columns
BLOCK = [((9, 17, 18), (1, -1, 1), 3), ((4, 8, 16), (-1, 1), 1), ((5, 9, 15), (1, -1), 2), ((13, 5, 20), (1, 1, -1), 2),
         ((1, 20, 7), (1, -1), 2), ((10, 1, 4), (-1, 1), 0), ((17, 25, 1), (1, -1), 4)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("shape,dirs,cap", BLOCK, ids=lambda v: str(v))
def test_block(libs, shape, dirs, cap, prec):
    g = workloads.rng(9)
    n = int(np.prod(shape))
    off = workloads.offsets(27)
    A = np.ascontiguousarray(workloads.random_sgdia(shape, 27, seed=10, block=3).reshape(27 * 9, n))
    D = np.ascontiguousarray(oracle.block_dinv(off, A, shape)).reshape(9, n)
    npt = np.float64 if prec == "fp64" else np.float32
    h = g.uniform(-1, 1, size=(len(dirs),) + shape + (3,)).astype(npt).astype(np.float64)
    a16 = sc = None
    Al = A.astype(npt)
    if prec == "fp16":
        sc = g.uniform(0.5, 2.0, size=(3, n)).astype(np.float32)
        half = A.astype(np.float16)
        a16 = half.view(np.uint16)
        Al = (half.astype(np.float32).reshape(27, 3, 3, n) * sc[None, :, None, :]).reshape(27 * 9, n)
    size = {"fp64": 8, "fp32": 4, "fp16": 2}[prec]
    for seed in (1, 2):
        x = np.empty_like(h)
        assert libs["block"].emu_block(size, ints(shape), len(dirs), ints(dirs), cap, C.c_ulong(seed), ptr(A), ptr(D),
                                       ptr(a16), ptr(sc), ptr(h), ptr(x)) == 0
        for k, d in enumerate(dirs):
            b = h[k].astype(npt)
            ref = oracle.bgs_sweep(off, Al, D.astype(npt), b, np.zeros_like(b), d, 1)
            assert np.array_equal(x[k].astype(npt), ref), (seed, k)


# columns around the block of 8 points, the wave of 64 and the longest column of the tiled kernel
LINE = [((9, 17, 16), 0), ((10, 9, 64), 2), ((9, 9, 7), 3), ((17, 20, 1), 3), ((5, 8, 65), 2), ((4, 5, 128), 2),
        ((3, 4, 129), 2), ((2, 3, 300), 3), ((1, 12, 8), 2), ((12, 1, 24), 2), ((16, 16, 33), 5)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("pat", [7, 19, 27])
@pytest.mark.parametrize("shape,cap", LINE, ids=lambda v: str(v))
def test_line(libs, shape, cap, pat, prec):
    off = workloads.offsets(pat)
    npt = np.float64 if prec == "fp64" else np.float32
    A = np.ascontiguousarray(workloads.random_sgdia(shape, pat, seed=11, symmetric=False).reshape(pat, -1))
    tr, tc = (np.ascontiguousarray(v, np.float64).ravel() for v in oracle.tri_factor(off, A, shape)[:2])
    f = workloads.rng(12).uniform(-1, 1, size=shape).astype(npt).astype(np.float64)
    Al, r, c, b = (v.astype(npt) for v in (A, tr, tc, f))
    u0 = oracle.lgs_sweep(off, Al, r, c, b, np.zeros(shape, npt), 1, 1)
    u1 = oracle.lgs_sweep(off, Al, r, c, b, u0, -1, 0)
    x = np.empty((2,) + shape)
    assert libs["line"].emu_line(8 if prec == "fp64" else 4, ints(shape), pat, cap, C.c_ulong(13), ptr(A), ptr(tr),
                                 ptr(tc), ptr(f), ptr(x)) == 0
    assert np.array_equal(x[0].astype(npt), u0)
    assert np.array_equal(x[1].astype(npt), u1)
