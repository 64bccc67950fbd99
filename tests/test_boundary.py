"""The C-ABI boundary without a GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments on the host before any HIP call."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "flashkmeans.h")
LIB = os.path.join(ROOT, "paper_2608_12629_amd", "libflashkmeans.so")

OK, EINVAL, EUNSUP, EWS, EHIP, ESCRATCH = 0, -1, -2, -3, -4, -5
SCRATCH_BYTES = 64 << 20
F32, BF16, F16 = 0, 1, 2


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kmeans_\w+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} not built (run __graft_entry__.build())")
    L = ctypes.CDLL(LIB)
    i64, i32, vp, sz = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t
    L.kmeans_workspace_bytes.argtypes = [i64, i64, i64, i64, i32]
    L.kmeans_workspace_bytes.restype = sz
    L.kmeans_assign.argtypes = [vp, i32, vp, i64, i64, i64, i64, vp, vp, vp, sz, vp]
    L.kmeans_update.argtypes = [vp, i32, vp, vp, i64, i64, i64, i64, vp, vp, vp, sz, vp]
    L.kmeans_lloyd.argtypes = [vp, i32, vp, i64, i64, i64, i64, i32, vp, vp, vp, vp, vp, sz, vp]
    L.kmeans_lloyd_noalloc.argtypes = [vp, i32, vp, i64, i64, i64, i64, i32, vp, vp, vp, vp, vp]
    L.kmeans_knn_workspace_bytes.argtypes = [i64, i64, i64, i64, i32, i32]
    L.kmeans_knn_workspace_bytes.restype = sz
    L.kmeans_knn.argtypes = [vp, vp, i32, i64, i64, i64, i64, i32, vp, vp, vp, sz, vp]
    L.kmeans_status_string.argtypes = [ctypes.c_int]
    L.kmeans_status_string.restype = ctypes.c_char_p
    return L


def test_header_declares_the_calls():
    assert declared_functions() == ["kmeans_assign", "kmeans_knn", "kmeans_knn_workspace_bytes",
                                    "kmeans_lloyd", "kmeans_lloyd_noalloc",
                                    "kmeans_status_string", "kmeans_update",
                                    "kmeans_workspace_bytes"]
    text = open(HEADER).read()
    assert re.search(r"#define KMEANS_SCRATCH_BYTES \(\(size_t\)64 << 20\)", text)


def test_every_declared_symbol_is_exported(lib):
    for name in declared_functions():
        assert hasattr(lib, name), name


def test_status_strings(lib):
    for st in (OK, EINVAL, EUNSUP, EWS, EHIP, ESCRATCH):
        s = lib.kmeans_status_string(st).decode()
        assert s and s != "unknown status"
    assert lib.kmeans_status_string(12345).decode() == "unknown status"


def test_workspace_bytes(lib):
    ws = lambda B, N, D, K, dt=BF16: lib.kmeans_workspace_bytes(B, N, D, K, dt)
    assert ws(1, 8_388_608, 128, 4096) > 0
    assert ws(1, 1000, 64, 10, F32) > 0
    # a workspace sized for N serves every smaller N (same B, D, K), on both
    # update paths (sorted: K = 1024; per-chunk partials: K = 64)
    for K in (1024, 64):
        prev = 0
        for N in (1, 100, 2048, 2049, 4096, 4097, 65536, 1 << 20):
            cur = ws(1, N, 128, K)
            assert cur >= prev
            prev = cur
    # the small-K one-hot path (16-bit, D = 64, K = 64)
    prev = 0
    for N in (1, 100, 2048, 2049, 4096, 65536, 1 << 20):
        cur = ws(2, N, 64, 64, F16)
        assert cur >= prev
        prev = cur
    # fp32 workgroups shrink for small problems (more of them): still monotone
    for D, K in ((64, 256), (128, 4096)):
        prev = 0
        for N in (1, 65536, 65537, 131071, 131072, 262143, 262144, 1 << 20):
            cur = ws(1, N, D, K, F32)
            assert cur >= prev, (D, K, N)
            prev = cur
    for K in (1, 7, 64, 1000, 4096, 32768, 65536):
        assert ws(1, 65536, 64, K) > 0
    assert ws(4, 1000, 64, 10) >= ws(1, 1000, 64, 10)
    # rejected shapes report 0
    assert ws(0, 10, 64, 4) == 0 and ws(1, 0, 64, 4) == 0 and ws(1, 10, 64, 0) == 0
    for D in (1, 3, 40, 100, 250, 272, 300, 2047):
        assert ws(1, 1000, D, 10) > 0, D    # served on zero-padded rows
    assert ws(1, 1000, 40, 10) > ws(1, 1000, 48, 10)  # plus the padded copies
    for D in (3, 17, 255):
        assert ws(1, 1000, D, 10, F32) > 0, D
    assert ws(1, 1000, 272, 10, F32) == 0   # fp32 rows past 256
    assert ws(1, 1000, 2049, 10) == 0
    for D in (16, 48, 96, 160, 208, 256, 288, 384, 640, 992, 2048):
        assert ws(1, 1000, D, 10) > 0, D    # 16-bit shapes in the domain
    for D in (16, 48, 80, 112, 128, 144, 256):
        assert ws(1, 1000, D, 10, F32) > 0, D
    assert ws(1, 10, 64, 70000) == 0        # K above the sort limit
    assert ws(1, 10, 64, 4, 7) == 0         # unknown dtype


FAKE = 0x10000          # a non-null, 16-byte-aligned address that is never dereferenced


def _assign(lib, X=FAKE, dt=BF16, C=FAKE, B=1, N=100, D=64, K=4, idx=FAKE, md=FAKE,
            ws=FAKE, wsb=1 << 40):
    return lib.kmeans_assign(X, dt, C, B, N, D, K, idx, md, ws, wsb, None)


def _update(lib, X=FAKE, dt=BF16, idx=FAKE, Cp=FAKE, B=1, N=100, D=64, K=4, Co=FAKE, n=FAKE,
            ws=FAKE, wsb=1 << 40):
    return lib.kmeans_update(X, dt, idx, Cp, B, N, D, K, Co, n, ws, wsb, None)


def _lloyd(lib, X=FAKE, dt=BF16, C=FAKE, B=1, N=100, D=64, K=4, iters=3, idx=FAKE, md=FAKE,
           n=FAKE, obj=None, ws=FAKE, wsb=1 << 40):
    return lib.kmeans_lloyd(X, dt, C, B, N, D, K, iters, idx, md, n, obj, ws, wsb, None)


@pytest.mark.parametrize("call", [_assign, _update, _lloyd])
def test_rejections_before_any_device_call(lib, call):
    assert call(lib, X=None) == EINVAL
    assert call(lib, X=FAKE + 4) == EINVAL          # misaligned
    assert call(lib, dt=3) == EINVAL
    assert call(lib, B=0) == EINVAL
    assert call(lib, N=0) == EINVAL
    assert call(lib, N=-5) == EINVAL
    assert call(lib, K=0) == EINVAL
    assert call(lib, D=0) == EINVAL
    assert call(lib, D=4096) == EUNSUP
    assert call(lib, D=2049) == EUNSUP
    assert call(lib, dt=F32, D=272) == EUNSUP  # fp32 rows up to 256
    assert call(lib, K=70000) == EUNSUP
    assert call(lib, N=1 << 31) == EUNSUP
    assert call(lib, ws=None) == EWS
    assert call(lib, wsb=16) == EWS


def test_specific_rejections(lib):
    assert _assign(lib, C=None) == EINVAL
    assert _assign(lib, idx=None) == EINVAL
    assert _assign(lib, md=None) == EINVAL
    assert _update(lib, idx=None) == EINVAL
    assert _update(lib, Cp=None) == EINVAL
    assert _update(lib, Co=None) == EINVAL
    assert _update(lib, n=None) == EINVAL
    assert _lloyd(lib, iters=0) == EINVAL
    assert _lloyd(lib, n=None) == EINVAL
    assert _lloyd(lib, obj=FAKE + 8) == EINVAL
    exact = lib.kmeans_workspace_bytes(1, 100, 64, 4, BF16)
    assert _assign(lib, wsb=exact - 1) == EWS


def _noalloc(lib, X=FAKE, dt=BF16, C=FAKE, B=1, N=100, D=64, K=4, iters=3, idx=FAKE, md=FAKE,
             n=FAKE, obj=None):
    return lib.kmeans_lloyd_noalloc(X, dt, C, B, N, D, K, iters, idx, md, n, obj, None)


def test_noalloc_rejections_before_any_device_call(lib):
    """The static-scratch entry point validates like kmeans_lloyd and rejects
    problems whose workspace exceeds the array, all before touching a GPU."""
    assert _noalloc(lib, X=None) == EINVAL
    assert _noalloc(lib, C=FAKE + 4) == EINVAL
    assert _noalloc(lib, n=None) == EINVAL
    assert _noalloc(lib, obj=FAKE + 8) == EINVAL
    assert _noalloc(lib, iters=0) == EINVAL
    assert _noalloc(lib, dt=3) == EINVAL
    assert _noalloc(lib, D=4096) == EUNSUP
    assert _noalloc(lib, K=70000) == EUNSUP
    # the 8M-point workload needs ~138 MiB of workspace: too big for the array
    assert lib.kmeans_workspace_bytes(1, 8_388_608, 128, 4096, BF16) > SCRATCH_BYTES
    assert _noalloc(lib, N=8_388_608, D=128, K=4096) == ESCRATCH
    # the largest N that fits, and the first that does not (fp32, D = 64, K = 256)
    fits = lambda N: lib.kmeans_workspace_bytes(1, N, 64, 256, F32) <= SCRATCH_BYTES
    lo, hi = 1, 1 << 28
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if fits(mid) else (lo, mid)
    assert _noalloc(lib, dt=F32, N=hi, D=64, K=256) == ESCRATCH
    assert fits(65536)   # the fp32 blob workload fits


def test_binding_refuses_without_library(tmp_path, monkeypatch):
    """The Python binding raises instead of falling back when the library is absent."""
    import importlib
    import paper_2608_12629_amd.kmeans as km
    monkeypatch.setattr(km, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(ImportError):
        km._load()
    importlib.reload(km)  # restore the module state with the real library


def _knn(lib, Q=FAKE, R=FAKE, dt=BF16, B=1, M=50, N=100, D=64, k=5, ni=FAKE, nd=FAKE, ws=FAKE,
         wsb=1 << 40):
    return lib.kmeans_knn(Q, R, dt, B, M, N, D, k, ni, nd, ws, wsb, None)


def test_knn_rejections(lib):
    assert _knn(lib, Q=None) == EINVAL
    assert _knn(lib, R=FAKE + 8) == EINVAL
    assert _knn(lib, ni=None) == EINVAL
    assert _knn(lib, nd=None) == EINVAL
    assert _knn(lib, k=0) == EINVAL
    assert _knn(lib, k=101) == EINVAL         # k > N
    assert _knn(lib, M=0) == EINVAL
    assert _knn(lib, dt=3) == EINVAL
    assert _knn(lib, dt=F32) == EUNSUP        # fp32 search not built
    assert _knn(lib, D=272) == EUNSUP
    assert _knn(lib, k=33) == EUNSUP
    assert _knn(lib, ws=None) == EWS
    assert _knn(lib, wsb=16) == EWS
    kw = lambda **a: lib.kmeans_knn_workspace_bytes(*[a.get(n, v) for n, v in
                                                      (("B", 1), ("M", 50), ("N", 100), ("D", 64),
                                                       ("k", 5), ("dt", BF16))])
    assert kw() > 0 and kw(k=33) == 0 and kw(dt=F32) == 0
    assert kw(N=1000) >= kw(N=100)


def _route(lib, B, M, N, D, k, dt=BF16, wsb=None):
    lib.fkm_knn_route.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_int, ctypes.c_size_t]
    return lib.fkm_knn_route(B, M, N, D, k, dt, 1 << 50 if wsb is None else wsb)


# us measured on an MI355X, bf16: the scan, the list kernel unsplit, in shares
# (0: never taken at that size)
@pytest.mark.parametrize("B,M,N,D,k,scan,whole,shares", [
    (1, 1, 64, 128, 10, 15, 38, 0), (1, 100, 1_000_003, 128, 10, 71, 15_730, 803),
    (1, 256, 300, 128, 10, 18, 74, 60), (1, 1024, 100_000, 128, 10, 98, 3175, 179),
    (1, 2048, 1_000_000, 128, 10, 776, 17_800, 994), (1, 4096, 300, 128, 32, 188, 193, 148),
    (4, 8, 1000, 32, 10, 17, 81, 48), (1, 512, 1_000_000, 32, 10, 93, 12_183, 664),
    (64, 2048, 64, 128, 1, 3106, 47, 0), (64, 2048, 64, 128, 10, 3470, 56, 0),
    (64, 2048, 300, 128, 10, 5858, 106, 103), (64, 1024, 64, 256, 10, 2050, 43, 0),
    (64, 1024, 300, 256, 10, 3445, 77, 0), (16, 2048, 64, 128, 10, 860, 41, 0),
    (64, 512, 1000, 128, 32, 4890, 330, 320), (16, 8192, 1000, 128, 32, 19_492, 1201, 1229),
    (16, 1024, 300, 256, 10, 871, 52, 92), (64, 2048, 3000, 32, 10, 1482, 298, 271),
    (1, 65_536, 1_048_576, 128, 10, 0, 18_291, 15_690), (1, 4096, 100_000, 32, 32, 152, 7512, 1142),
    (16, 4096, 300, 128, 10, 0, 77, 180), (16, 4096, 1000, 128, 10, 0, 134, 225),
    (64, 1024, 1000, 32, 10, 747, 129, 195), (4, 4096, 64, 256, 10, 506, 27, 79),
    (1, 256, 64, 256, 32, 16, 88, 109), (16, 1024, 300, 128, 32, 731, 186, 249),
])
def test_knn_route_is_the_fastest_measured(lib, B, M, N, D, k, scan, whole, shares):
    """The route takes at most a quarter more than the fastest of the three."""
    r = _route(lib, B, M, N, D, k)
    took = scan if r == 0 else whole if r == 1 else shares
    best = min(t for t in (scan, whole, shares) if t)
    assert took and took <= 1.25 * best, (r, took, best)


def test_knn_route_and_workspace(lib):
    """A search runs in any workspace that holds a copy of the rows: with less than the scan's
    maxima or the shares' lists need, by a route that fits."""
    full = lambda *a: lib.kmeans_knn_workspace_bytes(*a, BF16)
    for B, M, N, D, k in [(1, 100, 1_000_003, 128, 10), (1, 2048, 3000, 16, 32), (1, 40, 9_000, 40, 12),
                          (2, 2_100, 700, 24, 16), (1, 65_536, 1_048_576, 128, 10), (1, 30, 70, 16, 5)]:
        up = lambda v: (v + 255) // 256 * 256
        Np, Dk = (N + 127) // 128 * 128, (D + 15) // 16 * 16
        least = up(B * Np * Dk * 2) + up(B * Np * 4) + (up(B * M * Dk * 2) if Dk != D else 0)
        assert full(B, M, N, D, k) >= least
        assert _route(lib, B, M, N, D, k, wsb=least - 1) == -1
        assert _route(lib, B, M, N, D, k, wsb=least) >= 0
        assert _route(lib, B, M, N, D, k, wsb=full(B, M, N, D, k)) == _route(lib, B, M, N, D, k)
    assert _route(lib, 1, 10, 20, 64, 21) == -1 and _route(lib, 1, 10, 20, 64, 4, F32) == -1


@pytest.mark.parametrize("N,D,k", [(20_000, 32, 10), (50_000, 32, 16), (300_000, 32, 32), (130, 16, 5),
                                   (1_000_003, 128, 10), (70, 100, 1), (9_000, 200, 20)])
@pytest.mark.parametrize("B", [1, 3, 64])
def test_knn_workspace_grows_with_the_call(lib, B, N, D, k):
    """A workspace of the largest M or N serves every smaller one by the route that it
    would take with all the memory there is; beyond a copy of the rows it takes 64 MiB at most."""
    kw = lambda M, n: lib.kmeans_knn_workspace_bytes(B, M, n, D, k, BF16)
    up = lambda v: (v + 255) // 256 * 256
    queries = (1, 100, 128, 1024, 1025, 2048, 2049, 4096, 8192, 8193, 65_536, 131_072, 140_000, 700_000,
               1_500_000, 2_000_000)
    last = 0
    for M in queries:
        n = kw(M, N)
        assert n >= last, M
        last = n
        copy, Dk = up(B * (N + 127) // 128 * 128 * 2 * ((D + 15) // 16 * 16)), (D + 15) // 16 * 16
        padded = up(B * M * Dk * 2) + copy if Dk != D else 0
        assert n <= up(B * (N + 127) * 4) + padded + B * 128 * Dk * 2 + max(copy, 64 << 20) + 8192, M
        assert _route(lib, B, M, N, D, k, wsb=kw(queries[-1], N)) == _route(lib, B, M, N, D, k), M
    last = 0
    for n in sorted({k, 64, 300, 1000, 16_384, 100_000, 262_144, 262_145, 524_288, 524_289, 2_000_000, N}):
        if n >= k:
            assert kw(1500, n) >= last, n
            last = kw(1500, n)


def test_calibration_library_exports_its_header():
    """libfkm_calib.so (the benchmark's in-run ceilings) exports every call that
    include/fkm_calib.h declares and rejects bad arguments on the host."""
    path = os.path.join(ROOT, "paper_2608_12629_amd", "libfkm_calib.so")
    if not os.path.exists(path):
        pytest.fail(f"{path} not built (run __graft_entry__.build())")
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "fkm_calib.h")).read(),
                  flags=re.S)
    names = sorted(set(re.findall(r"\b(fkm_calib_\w+)\s*\(", text)))
    assert names == ["fkm_calib_gather", "fkm_calib_mfma", "fkm_calib_read"]
    L = ctypes.CDLL(path)
    for n in names:
        assert hasattr(L, n), n
    vp, i32, i64, sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_size_t
    L.fkm_calib_mfma.argtypes = [vp, i32, i32, vp]
    L.fkm_calib_read.argtypes = [vp, sz, vp, i32, vp]
    L.fkm_calib_gather.argtypes = [vp, i64, i32, vp, i64, vp, i32, vp]
    assert L.fkm_calib_mfma(None, 512, 10, None) == -1
    assert L.fkm_calib_mfma(FAKE, 0, 10, None) == -1
    assert L.fkm_calib_read(FAKE, 17, FAKE, 16, None) == -1        # not whole 16-byte chunks
    assert L.fkm_calib_read(FAKE + 4, 16, FAKE, 16, None) == -1    # misaligned
    assert L.fkm_calib_gather(FAKE, 10, 2048, FAKE, 10, FAKE, 16, None) == -1  # rows > 1 KiB
    assert L.fkm_calib_gather(FAKE, 0, 256, FAKE, 10, FAKE, 16, None) == -1
