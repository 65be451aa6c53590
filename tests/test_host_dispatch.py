"""The library's host side without a GPU: which kernels a call launches with
which grids, what scratch it asks for, and what it does when the runtime refuses
something.  Each check runs in a child process whose HIP runtime is the recorder
of tests/hip_record/ (nothing is computed; device pointers are never read)."""
import json
import os
import shutil
import subprocess
import sys

import pytest

from tests.decode_forms import FORMS

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
REC = os.path.join(HERE, "hip_record")

PRELUDE = """
import ctypes, importlib.util, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
rec.rec_malloc_limit.argtypes = [ctypes.c_uint64]
spec = importlib.util.spec_from_file_location("mvk_lib", sys.argv[2])
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
lib = L.load(int(sys.argv[3]))
assert any(sys.argv[1] in l for l in open("/proc/self/maps"))
next_ptr = [1 << 40]
def ptr():  # an aligned device address that nothing reads
    next_ptr[0] += 1 << 36
    return next_ptr[0]
def code(k, r): return L.MvkCode(k, r, ptr(), ptr(), ptr(), ptr())
def key(m, n, rx, ry): return L.MvkKey(m, n, code(n, rx), code(m, ry), ptr(), ptr())
def sparse(count, t): return L.MvkSparse(ptr(), ptr(), t, count)
def launches():
    out = []
    for i in range(rec.rec_count()):
        g = (ctypes.c_uint32 * 3)()
        rec.rec_grid(i, g)
        out.append([rec.rec_name(i).decode().replace("void ", "").replace("mvk::(anonymous namespace)::", "").split("(")[0],
                    g[0], g[1]])
    return out
ref = ctypes.byref
result = {}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("hip_record")
    so = str(d / "libamdhip64.so.7")
    r = subprocess.run([cxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                        f"-Wl,--version-script={REC}/hip_record.map", "-o", so, f"{REC}/hip_record.cpp"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = os.path.join(ROOT, "paper_2609_10264_amd", "_lib.py")

    def run(body, p=2**31 - 1):
        if not os.path.exists(os.path.join(ROOT, "paper_2609_10264_amd", "libmvk.so")):
            pytest.skip("libmvk.so not built")
        r = subprocess.run([sys.executable, "-c", PRELUDE + body + "\nprint(json.dumps(result))\n", so, lib, str(p)],
                           capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout.splitlines()[-1])

    return run


# Short syndromes join the long ones only while all of them fit one sequence of
# launches (65535 vectors): 65533 long noise vectors and two short challenges do,
# 65534 and 65535 do not, and the call must go on as two launches.
@pytest.mark.parametrize("B", [65533, 65534, 65535])
def test_prepare_most_columns(host, B):
    out = host(f"""
k = key(16, 16400, 2, 2)
ex, ey = sparse({B}, 8), sparse(2, 8)
result["st"] = lib.mvk_client_prepare(ref(k), ref(ex), ref(ey), ptr(), ptr(), ptr(), ptr(), None, 0, None)
result["launches"] = launches()
""")
    assert out["st"] == 0
    names = [l[0] for l in out["launches"]]
    assert any(n.startswith("client_prepare_kernel") for n in names) == (B > 65533), names
    assert sum(n.startswith("syn_p1") for n in names) == 1 and sum("syn_p3" in n for n in names) == 1


# keygen where the workspace cannot hold the segmented encoding (a nearly full
# card; a stream that captures and has had a smaller workspace): the form that
# needs m*n + max(Nx*m, Ny*n)*4 bytes and 1/32 (the segment sums) takes its place.
@pytest.mark.parametrize("how", ["full", "capture"])
def test_keygen_scratch(host, how):
    out = host(f"""
m, n, r = 2049, 8192, 3
k = key(m, n, r, r)
need = int((m * n + 4 * r * m * n) * 1.034)
if {how!r} == "full":
    rec.rec_malloc_limit(need)
else:
    # 2N + (segments + 1) * 2 words of workspace per vector: 2 vectors of N = need / 16
    N = need // 16
    assert lib.mvk_raa_syndrome(ref(code(N, 1)), ptr(), 2, ptr(), None) == 0
    rec.rec_reset()
    rec.rec_capture(1)
result["st"] = lib.mvk_keygen(ref(k), ptr(), None)
result["launches"] = launches()
rec.rec_reset()
result["free"] = lib.mvk_keygen(ref(k), ptr(), None)
result["then"] = launches()
""")
    assert out["st"] == 0 and out["free"] == 0
    assert [l[0] for l in out["launches"] if "fill" not in l[0]][1].startswith("enc_pass1")
    assert any(l[0].startswith("enc_seg") for l in out["then"])


# client_prepare where the workspace cannot hold the short syndromes beside the
# long ones: they keep their own launch, which needs none.
@pytest.mark.parametrize("call", ["one", "group", "multi"])
@pytest.mark.parametrize("how", ["full", "capture"])
def test_prepare_scratch(host, call, how):
    out = host(f"""
m, n, B, call = 8190, 9000, 64, {call!r}  # N = 16380 (short), 18000 (long)
k = key(m, n, 2, 2)
ex, ey = sparse(B, 8), sparse(16, 8)
def run():
    mx, my, r, u = ptr(), ptr(), ptr(), ptr()
    if call == "one":
        return lib.mvk_client_prepare(ref(k), ref(ex), ref(ey), mx, my, r, u, None, 0, None)
    P1 = lambda a: (ctypes.c_void_p * 1)(a)
    S1 = lambda a: (ctypes.POINTER(type(a)) * 1)(ctypes.pointer(a))
    keys, eys = S1(k), S1(ey)
    if call == "group":
        return lib.mvk_client_prepare_group(1, keys, ref(ex), eys, mx, P1(my), P1(r), P1(u), None, 0, None)
    return lib.mvk_client_prepare_multi(1, keys, S1(ex), eys, P1(mx), P1(my), P1(r), P1(u), None, 0, None)
# the long vectors' work arrays, and 1 MiB for everything else
rec.rec_malloc_limit(B * (2 * 18000 * 4 + 152) + (1 << 20))
if {how!r} == "capture":  # the call before sizes the workspace
    assert run() == 0
    rec.rec_reset()
    rec.rec_capture(1)
result["st"] = run()
result["launches"] = launches()
rec.rec_reset()
result["free"] = run()
result["then"] = launches()
""")
    assert out["st"] == 0 and out["free"] == 0, out
    assert any(l[0].startswith("client_prepare_kernel") for l in out["launches"])
    assert not any(l[0].startswith("client_prepare_kernel") for l in out["then"])


# batch_verify likewise: the short code's syndromes in their own launch.
@pytest.mark.parametrize("how", ["full", "capture"])
def test_batch_scratch(host, how):
    out = host(f"""
m, n, B, ell = 9000, 1000, 8, 16  # N = 18000 (long), 16000 (short)
cy, c2 = code(m, 2), code(B * n, 2)
e, e2 = sparse(ell, 8), sparse(ell, 8)
run = lambda: lib.mvk_batch_verify(ref(cy), ref(c2), ptr(), m, n, B, ptr(), ptr(), ref(e), ptr(), ref(e2), None, None,
                                   None, None, ptr(), None)
need = ell * (2 * 18000 * 4 + 152) + 4 * ell * (m + B * n) + (1 << 20)
rec.rec_malloc_limit(need)
if {how!r} == "capture":  # the call before sizes the workspace
    assert run() == 0
    rec.rec_reset()
    rec.rec_capture(1)
result["st"] = run()
result["launches"] = launches()
rec.rec_reset()
result["free"] = run()
result["then"] = launches()
""")
    assert out["st"] == 0 and out["free"] == 0, out
    assert any(l[0].startswith("syn_wg") for l in out["launches"])
    assert not any(l[0].startswith("syn_wg") for l in out["then"])


# decode/verify of a long block whose second launch is refused: the first has
# added to accumulators that the second would have cleared, so they are cleared
# before the call returns (else the next verification on the stream rejects).
def test_refused_second_launch_leaves_no_sums(host):
    out = host("""
k = key(16400, 300, 2, 2)
ex, ey = sparse(2, 8), sparse(2, 8)
rec.rec_refuse_launch(2)  # after the fill of the new control region and the first launch
result["st"] = lib.mvk_decode_verify(ref(k), ptr(), ptr(), 2, ref(ex), ref(ey), ptr(), None, None, ptr(), None)
result["launches"] = launches()
""")
    assert out["st"] == -4
    names = [l[0].split("<")[0] for l in out["launches"]]
    assert names == ["fill_u32", "decode_verify_long1", "refused", "fill_u32"]


# k-ranges of the digits-stationary kernel (5 to 16 queries): none where a row is
# one chunk of eight k-blocks, four (not eight, which would split a chunk) at 2048
# x 2048 with 8 queries, and the ranges that few row blocks take.
@pytest.mark.parametrize("m,n,B,ks", [
    (1024, 512, 16, 1), (1024, 512, 8, 1), (6000, 512, 16, 1), (2048, 2048, 8, 4), (3072, 2048, 5, 4), (2048, 2048, 16, 4),
    (1024, 4096, 16, 8), (4096, 4096, 8, 8), (4096, 4096, 16, 8), (11008, 4096, 16, 2), (8192, 3072, 16, 4), (28672, 1000, 8, 1),
])
def test_k_ranges(host, m, n, B, ks):
    out = host(f"""
result["st"] = lib.mvk_server_eval_packed(ptr(), {m}, {n}, ptr(), {B}, ptr(), None)
result["launches"] = launches()
""")
    name, grid, _ = out["launches"][-1]
    assert out["st"] == 0 and name.startswith("server_eval_mfma_dstat<%d, 1," % (2 if B <= 8 else 4)), name
    blocks = -(-m // 128)
    assert grid == -(-blocks // (8 // ks)) * 8


@pytest.mark.parametrize("m,ry,B,ell,ty,inplace,kernel", FORMS)
def test_decode_forms(host, m, ry, B, ell, ty, inplace, kernel):
    # (a compute unit's LDS holds two workgroups of the second tile size, one of the larger ones)
    out = host(f"""
rec.rec_occupancy({2 if ry * m <= 8192 else 1})
k = key({m}, 64, 2, {ry})
ex, ey = sparse({B}, 9), sparse({ell}, {ty})
yh = ptr()
result["st"] = lib.mvk_decode_verify(ref(k), ptr(), yh, {B}, ref(ex), ref(ey), yh if {inplace} else ptr(), None, None,
                                     ptr(), None)
result["launches"] = launches()
""")
    assert out["st"] == 0
    assert out["launches"][-1][0].startswith(kernel), out["launches"]


# verify alone: the rule on many columns holds with r = 2 only
@pytest.mark.parametrize("m,ry,B,ell,kernel", [(4096, 2, 16, 2, "decode_verify_syn<16, 4>"),
                                               (4096, 2, 16, 3, "decode_verify_dot<16, 16>"),
                                               (5000, 1, 16, 1, "decode_verify_dot<16, 16>")])
def test_verify_forms(host, m, ry, B, ell, kernel):
    out = host(f"""
rec.rec_occupancy(2)
k = key({m}, 64, 2, {ry})
result["st"] = lib.mvk_verify(ref(k), ptr(), ptr(), {B}, ref(sparse({ell}, 31)), None, None, ptr(), None)
result["launches"] = launches()
""")
    assert out["st"] == 0 and out["launches"][-1][0].startswith(kernel), out["launches"]


# More segments than the chip holds workgroups: four stripes each, also of dense
# vectors (the sizes of the GPU test).
@pytest.mark.parametrize("k,r,count,stripes", [(8500, 2, 13, 1), (8500, 2, 120, 1), (8500, 2, 125, 4), (20500, 1, 110, 4)])
def test_dense_stripes(host, k, r, count, stripes):
    out = host(f"""
result["st"] = lib.mvk_raa_syndrome(ref(code({k}, {r})), ptr(), {count}, ptr(), None)
result["launches"] = launches()
""")
    assert out["st"] == 0
    assert [l[0] for l in out["launches"][1:]] == [f"syn_p1<false, {stripes}>", f"syn_p2<{stripes}>", "syn_p3"]


# keygen with rows that are not whole 16-byte granules: the offsets of the segments
# are a product that reads the matrix once for 16, 8 or 4 of its 62 queries
# (rows up to 16384, 32768 and above), which pays up to 4 r readings.
@pytest.mark.parametrize("m,n,r,forms", [
    (2051, 65537, 1, ["enc_pass2"]), (2051, 33001, 2, ["enc_pass2", "enc_seg<false>"]), (2051, 33001, 4, ["enc_seg<false>"]),
    (4099, 30001, 1, ["enc_pass2", "enc_seg<false>"]), (2051, 30001, 2, ["enc_seg<false>"]),
    (40001, 3001, 1, ["enc_pass2"]), (40001, 3001, 2, ["enc_seg<false>", "enc_pass2"]), (2051, 131056, 2, ["enc_seg<false>"]),
])
def test_keygen_long_ragged_rows(host, m, n, r, forms):
    out = host(f"""
k = key({m}, {n}, {r}, {r})
result["st"] = lib.mvk_keygen(ref(k), ptr(), None)
result["launches"] = launches()
""")
    assert out["st"] == 0
    names = [n for n, _, _ in out["launches"] if n.startswith(("enc_pass2", "enc_seg<false>"))]
    names = ["enc_pass2" if n.startswith("enc_pass2") else n for n in names]
    assert [n for i, n in enumerate(names) if names[i - 1:i] != [n]] == forms


# Long syndromes placed by XCD (whole eights and a rest of six or more; grid.y counts
# the empty places): vectors of one length, not 20 short ones with two long ones
# that two XCDs would have to take by themselves.
@pytest.mark.parametrize("m,n,ry,B,ell,rows", [(64, 9000, 2, 22, 0, 24), (64, 9000, 2, 21, 0, 21), (17152, 81, 4, 20, 2, 22),
                                               (17152, 81, 4, 6, 16, 24), (9000, 17152, 2, 20, 2, 24)])
def test_placement_by_xcd(host, m, n, ry, B, ell, rows):
    out = host(f"""
k = key({m}, {n}, 2, {ry})
ex, ey = sparse({B}, 8), sparse({ell}, 8)
result["st"] = lib.mvk_client_prepare(ref(k), ref(ex), ref(ey) if {ell} else None, ptr(), ptr(), ptr(), ptr(), None, 0, None)
result["launches"] = launches()
""")
    assert out["st"] == 0
    assert [l[2] for l in out["launches"] if l[0].startswith("syn_p1")] == [rows], out["launches"]


# ... nor where the longest vector would leave most of the joined grid empty
@pytest.mark.parametrize("m,n,rx,ry,B,ell,join", [(23168, 563, 4, 8, 37, 2, False), (13248, 1212, 1, 8, 42, 4, True),
                                                     (8500, 64, 2, 2, 254, 2, True), (8500, 64, 2, 2, 257, 2, False),
                                                     (16400, 64, 2, 2, 254, 2, False)])
def test_prepare_join_of_uneven_lengths(host, m, n, rx, ry, B, ell, join):
    out = host(f"""
k = key({m}, {n}, {rx}, {ry})
ex, ey = sparse({B}, 8), sparse({ell}, 8)
result["st"] = lib.mvk_client_prepare(ref(k), ref(ex), ref(ey), ptr(), ptr(), ptr(), ptr(), None, 0, None)
result["launches"] = launches()
""")
    assert out["st"] == 0
    assert any(l[0].startswith("client_prepare_kernel") for l in out["launches"]) == (not join), out["launches"]
