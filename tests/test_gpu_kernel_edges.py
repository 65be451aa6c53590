"""GPU parity at the edges of the kernels' ranges (tile remainders, the smallest
and largest sizes of a dispatch rule, alignments), against the CPU oracle.
Every value is an integer mod p: all comparisons are exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_10264_amd as mvk
import synth
from tests.decode_forms import FORMS
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


# Row-major W whose rows are not whole aligned 16-byte granules: below 16 bytes
# in all; one 16-byte load moved down from every row (n < 16); the end of the
# matrix in a full and in a partial row tile; 4 | 5 queries (small |
# digits-stationary kernel), 8 | 9 digit tiles, 16 | 17 and more than one group
# of 16; row lengths around one k-block and around a k split; the longest
# rows of the digits-stationary kernel (16384) and one more.
@pytest.mark.parametrize("m,n,B,off", [
    (1, 7, 3, 1), (3, 5, 6, 0), (2, 8, 5, 3), (5, 3, 9, 2), (16, 1, 5, 0), (129, 17, 4, 0), (128, 63, 5, 0),
    (127, 65, 8, 5), (257, 127, 9, 0), (130, 1001, 16, 1), (64, 4095, 17, 0), (500, 3001, 12, 0), (33, 4096, 16, 8),
    (31, 2047, 40, 0), (150, 16383, 16, 0), (20, 16384, 9, 7), (20, 16385, 9, 0), (40, 32767, 8, 0), (17, 33001, 6, 0),
])
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_row_major_any_alignment(m, n, B, off, p):
    W = synth.weights(500 + m + n, m, n, lo=-128)
    X = synth.field_uniform(501 + B + n, (B, n), p=p)
    buf = torch.full((off + m * n + 16,), 0x55, dtype=torch.int8, device="cuda")
    dW = buf[off:off + m * n].view(m, n)
    dW.copy_(dev(W))
    print("row-major", m, n, B, off, p, flush=True)
    assert np.array_equal(host(mvk.server_eval(dW, dev(X), p=p)), oracle.server_eval(W, X, p=p))


# Query rows at any word alignment on packed W (the wide loads of X).
@pytest.mark.parametrize("m,n,B", [(40, 4099, 1), (200, 1001, 3), (200, 4099, 12), (300, 999, 33), (24600, 130, 20)])
def test_query_alignment(m, n, B):
    W = synth.weights(520 + m + n, m, n)
    X = synth.field_uniform(521 + B + n, (B, n))
    buf = torch.zeros((B * n + 3,), dtype=torch.int32, device="cuda")
    for off in (0, 1, 3):
        dX = buf[off:off + B * n].view(B, n)
        dX.copy_(dev(X))
        assert np.array_equal(host(mvk.server_eval(mvk.pack_weights(dev(W)), dX)), oracle.server_eval(W, X))



# The end of a query row in the wide loads of X: rows of fewer than four elements, of
# every remainder by four and by sixteen, and the last row at the end of its buffer.
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 15, 17, 18, 31, 63, 65, 130, 179, 999, 4097, 4102])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 7, 12, 16, 20, 40])
def test_query_row_ends(n, B):
    m = 37
    W = synth.weights(530 + n, m, n, lo=-128)
    X = synth.field_uniform(531 + B + n, (B, n))
    print("row ends", n, B, flush=True)
    want = oracle.server_eval(W, X)
    buf = torch.full((B * n + 8,), -1, dtype=torch.int32, device="cuda")  # (what a read past a row would bring in)
    for off in (0, 5):
        dX = buf[off:off + B * n].view(B, n)
        dX.copy_(dev(X))
        for dW in (dev(W), mvk.pack_weights(dev(W))):
            assert np.array_equal(host(mvk.server_eval(dW, dX)), want)


# keygen with the segment offsets from one server product (at least 2048 vectors
# and 192 MB of intermediate sums, 400 MB where the matrix rows are not whole
# 16-byte granules): the fewest vectors, both encodings; an odd number of
# vectors (the last lane takes the last four) with a ragged last segment, next
# to Q on the three-pass form; odd row lengths on both sides; one vector too few.
@pytest.mark.parametrize("m,n,rx,ry", [(2048, 8192, 3, 3), (2051, 6400, 4, 4), (2049, 16387, 4, 3), (2047, 8192, 3, 2)])
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_keygen_segments(m, n, rx, ry, p):
    from tests.gpu_util import code
    print("keygen", m, n, rx, ry, p, flush=True)
    W = synth.weights(540 + m + n, m, n, lo=-128)
    cx, cy = synth.raa_code(541 + n, n, rx, p=p), synth.raa_code(542 + m, m, ry, p=p)
    key = mvk.keygen(mvk.Key.allocate(m, n, code(cx, p), code(cy, p)), dev(W))
    PT, Q = oracle.keygen(W, cx, cy, p=p, nthreads=oracle.threads())
    assert np.array_equal(host(key.PT), PT)
    assert np.array_equal(host(key.Q), Q)



# Long syndromes of dense vectors: one vector's segments on one XCD (six vectors and
# more; an empty place at seven, vectors left over at 13), and four stripes a
# workgroup (more than 2048 segments; a last one that is cut short).
@pytest.mark.parametrize("k,r,count", [(4200, 4, 7), (8500, 2, 13), (8500, 2, 125), (20500, 1, 110)])
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_dense_syndromes_many_vectors(k, r, count, p):
    from tests.gpu_util import code
    print("dense syndromes", k, r, count, p, flush=True)
    c = synth.raa_code(640 + k, k, r, p=p)
    v = synth.field_uniform(641 + k, (count, k * r), p=p)
    got = host(mvk.raa_syndrome(code(c, p), dev(v)))
    for i in range(count):
        assert np.array_equal(got[i], oracle.syn(c, v[i], p=p))


# Preparations whose gathers take their own launch: many columns of a short
# matrix, where items of 1024 columns would no longer need that launch; short
# syndromes that join long ones (up to 256 of them, and one more); the gathers
# beside the second pass of long ones (one stripe per workgroup), by items of 64,
# 256 and 1024 columns; four stripes.  (With 16400 rows the joined grid would be
# mostly empty, with 8500 not.)
@pytest.mark.parametrize("m,n,rx,ry,B,tx", [(1024, 64, 2, 2, 300, 8), (8192, 300, 3, 3, 40, 20), (4352, 6000, 3, 2, 62, 70),
                                            (16400, 64, 2, 2, 254, 8), (16400, 64, 2, 2, 260, 8),
                                            (8191, 300, 3, 3, 40, 20), (1100, 8200, 2, 2, 220, 8),
                                            (8500, 64, 2, 2, 254, 8), (8500, 64, 2, 2, 257, 8)])
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_prepare_split(m, n, rx, ry, B, tx, p):
    from tests.gpu_util import Instance
    print("prepare", m, n, rx, ry, B, tx, p, flush=True)
    t = Instance(600 + m + B, m, n, B, rx, tx, 31, 2, ry=ry, p=p)
    t.to_device()
    mvk.keygen(t.key, t.dW)
    prep = mvk.client_prepare(t.key, t.dexi, t.dexv, t.deyi, t.deyv)
    zero = np.zeros((B, n), dtype=np.uint32)
    Mx = oracle.encode(t.cx, zero, t.exi, t.exv, p=p)
    assert np.array_equal(host(prep.Mx), Mx)
    assert np.array_equal(host(prep.My), oracle.server_eval(t.W, Mx, p=p, nthreads=oracle.threads()))
    R = oracle.encode(t.cy, np.zeros((2, m), dtype=np.uint32), t.eyi, t.eyv, p=p)
    assert np.array_equal(host(prep.R), R)
    assert np.array_equal(host(prep.U), oracle.server_eval(np.ascontiguousarray(t.W.T), R, p=p))


# Decode/verify without r_q (up to 4 repetitions; blocks up to 16384 positions: 64
# terms and 16 columns, 8 up to 4096 positions; long ones: 4 columns and 8 sums):
# no noise, the most terms, columns and repetitions and one more of each; N around
# one segment of 512 and of 1024 positions, 16384 (the last block of one
# workgroup) and one more; Y over Yhat.
@pytest.mark.parametrize("m,n,rx,ry,B,tx,ty,ell,inplace", [
    (1, 1, 1, 1, 1, 0, 1, 1, False), (5, 3, 2, 3, 3, 6, 15, 4, False), (256, 256, 2, 2, 1, 8, 31, 2, False),
    (257, 300, 2, 2, 8, 64, 64, 2, False), (171, 100, 3, 3, 2, 65, 65, 3, False), (1000, 700, 3, 4, 4, 128, 64, 2, False),
    (500, 500, 3, 1, 1, 192, 64, 1, False), (300, 500, 2, 3, 5, 20, 31, 4, False), (300, 500, 2, 3, 9, 20, 31, 2, False),
    (300, 500, 2, 3, 2, 20, 31, 5, False), (300, 500, 2, 3, 2, 20, 31, 2, True), (4097, 200, 3, 1, 16, 9, 31, 4, False),
    (4097, 200, 3, 1, 17, 9, 31, 2, False), (4096, 200, 3, 4, 9, 63, 63, 2, False), (4096, 200, 3, 1, 8, 63, 63, 2, False),
    (4097, 200, 3, 4, 1, 63, 63, 2, False), (5462, 4097, 4, 3, 4, 40, 31, 2, False), (5462, 500, 4, 4, 3, 40, 31, 3, False),
    (8192, 5000, 4, 8, 2, 154, 200, 4, False), (8192, 5000, 4, 8, 8, 154, 200, 4, False), (5000, 300, 2, 4, 5, 9, 31, 1, False),
    (9001, 300, 2, 2, 2, 30, 31, 2, True), (16384, 1000, 3, 8, 4, 8, 31, 2, False),
])
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_few_terms_few_columns(m, n, rx, ry, B, tx, ty, ell, inplace, p):
    from tests.gpu_util import Instance
    print("decode", m, n, rx, ry, B, tx, ty, ell, inplace, p, flush=True)
    t = Instance(560 + m + ty, m, n, B, rx, tx, ty, ell, ry=ry, p=p)
    t.to_device()
    mvk.keygen(t.key, t.dW)
    xh = mvk.encode(t.key, t.dX, t.dexi, t.dexv)
    assert np.array_equal(host(xh), oracle.encode(t.cx, t.X, t.exi, t.exv, p=p))
    yh = mvk.server_eval(t.dW, xh, p=p)
    yh[B - 1, m - 1] = (yh[B - 1, m - 1].long() + 1).remainder(p).int()  # the last column is wrong
    hyh = host(yh)
    PT, Q = host(t.key.PT), host(t.key.Q)
    acc0, vL0, vR0 = oracle.verify(t.cy, Q, host(xh), hyh, t.eyi, t.eyv, p=p)
    for _ in range(2):  # the control region is left as it was found
        out = yh.clone()
        vL = torch.empty((ell, B), dtype=torch.int32, device="cuda")
        vR = torch.empty_like(vL)
        Y, acc, _, _ = mvk.decode_verify(t.key, xh, out, t.dexi, t.dexv, t.deyi, t.deyv, Y=out if inplace else None,
                                         vL=vL, vR=vR)
        assert np.array_equal(host(vL), vL0) and np.array_equal(host(vR), vR0)
        assert host(acc).tolist() == acc0.astype(np.uint32).tolist()
        assert np.array_equal(host(Y), oracle.decode(PT, hyh, t.exi, t.exv, p=p))



# Every form of decode_verify up to 16384 positions, each with an honest response
# and one with the first column tampered.
@pytest.mark.parametrize("m,ry,B,ell,ty,inplace,kernel", FORMS)
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_decode_forms(m, ry, B, ell, ty, inplace, kernel, p):
    from tests.gpu_util import Instance
    print("decode form", m, ry, B, ell, ty, inplace, kernel, p, flush=True)
    t = Instance(580 + m + ty, m, 64, B, 2, 9, ty, ell, ry=ry, p=p).to_device()
    mvk.keygen(t.key, t.dW)
    PT, Q = host(t.key.PT), host(t.key.Q)
    xh = mvk.encode(t.key, t.dX, t.dexi, t.dexv)
    hyh = oracle.server_eval(t.W, host(xh), p=p)
    for wrong in (0, 1):
        hyh[0, m - 1] = (int(hyh[0, m - 1]) + wrong) % p
        yh = dev(hyh)
        vL = torch.empty((ell, B), dtype=torch.int32, device="cuda")
        vR = torch.empty_like(vL)
        Y, acc, _, _ = mvk.decode_verify(t.key, xh, yh, t.dexi, t.dexv, t.deyi, t.deyv, Y=yh if inplace else None,
                                         vL=vL, vR=vR)
        oacc, ovL, ovR = oracle.verify(t.cy, Q, host(xh), hyh, t.eyi, t.eyv, p=p)
        assert host(acc).tolist() == oacc.astype(np.uint32).tolist() == [1 - wrong] + [1] * (B - 1)
        assert np.array_equal(host(vL), ovL) and np.array_equal(host(vR), ovR)
        assert np.array_equal(host(Y), oracle.decode(PT, hyh, t.exi, t.exv, p=p))


# Eight k-ranges of the digits-stationary kernel where there are few row blocks:
# ranges that are empty or cut short, one row, the last row block of that rule.
@pytest.mark.parametrize("m,n,B", [(1, 300, 5), (100, 577, 16), (256, 4096, 8), (256, 4096, 16), (1000, 4100, 12),
                                   (2048, 2048, 16), (4096, 4096, 8), (8064, 640, 9)])
@pytest.mark.parametrize("p", [synth.P, synth.P_BABYBEAR])
def test_many_k_ranges(m, n, B, p):
    W = synth.weights(700 + m + n, m, n, lo=-128)
    X = synth.field_uniform(701 + B + n, (B, n), p=p)
    print("k-ranges", m, n, B, p, flush=True)
    want = oracle.server_eval(W, X, p=p, nthreads=oracle.threads())
    for dW in (dev(W), mvk.pack_weights(dev(W))):
        for _ in range(2):
            assert np.array_equal(host(mvk.server_eval(dW, dev(X), p=p)), want)


# Batch verification with one long and one short code (both by segments), odd
# numbers of repetitions, and more sums than threads in the last workgroup.
@pytest.mark.parametrize("m,n,B,ell,ell2", [(300, 2100, 4, 2, 2), (5500, 70, 3, 3, 1), (300, 2100, 4, 1, 5), (20, 30, 86, 3, 4)])
def test_batch_long_and_short_code(m, n, B, ell, ell2):
    cy, c2 = synth.raa_code(620 + m, m, 3), synth.raa_code(621 + n, B * n, 2)
    from tests.gpu_util import code
    Ws = [synth.weights(622 + b, m, n) for b in range(B)]
    X = synth.field_uniform(630, (B, n))
    ei, ev = synth.sparse(631, ell, cy["N"], 31)
    e2i, e2v = synth.sparse(632, ell2, c2["N"], 31)
    one = synth.raa_code(633, n, 2)
    Qs = [mvk.keygen(mvk.Key.allocate(m, n, code(one), code(cy)), dev(W)).Q for W in Ws]
    QtT, Qaux = mvk.batch_preprocess(Qs, code(c2))
    Y = np.concatenate([oracle.server_eval(W, X[b:b + 1]) for b, W in enumerate(Ws)])
    Y[B - 1, m - 1] = (int(Y[B - 1, m - 1]) + 1) % synth.P
    ut = mvk.batch_project(QtT, n, dev(ei), dev(ev))
    out = [torch.empty((ell, k), dtype=torch.int32, device="cuda") for k in (B, B, ell2, ell2)]
    acc = mvk.batch_verify(code(cy), code(c2), Qaux, dev(X), dev(Y), dev(ei), dev(ev), ut, dev(e2i), dev(e2v),
                           vL=out[0], vR=out[1], sL=out[2], sR=out[3])[0]
    hQ = [host(Q) for Q in Qs]
    oacc, _, *want = oracle.batch_verify(cy, c2, oracle.batch_aux(hQ, c2), X, Y, ei, ev,
                                         oracle.batch_project(hQ, ei, ev), e2i, e2v)
    assert host(acc).tolist() == oacc.astype(np.uint32).tolist() == [1] * (B - 1) + [0]
    for got, w in zip(out, want):
        assert np.array_equal(host(got), w)
