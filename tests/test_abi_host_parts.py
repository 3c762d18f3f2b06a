"""The entry points of tmamba_parts.h and tmamba_decode16.h on the host: every
declared symbol is exported and bound, and bad arguments are rejected with the
documented status codes before any launch.  No test here passes arguments that
would reach a kernel launch."""

import ctypes
import os
import re

import pytest

from paper_2606_18114_amd import ops

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EINVAL, ESHAPE, EALIGN = 1, 2, 3
P = 0x7F0000000000  # a 4 KiB-aligned fake device address, never dereferenced
BOUND = {"tmamba_parts.h": ops.SIGNATURES_PARTS, "tmamba_decode16.h": ops.SIGNATURES_DECODE16}


@pytest.fixture(scope="module")
def L():
    # TM_ABI_TEST_LIB: the host-only sanitizer build (tests/test_abi_sanitized.py)
    alt = os.environ.get("TM_ABI_TEST_LIB")
    if alt:
        lib = ctypes.CDLL(alt)
        for sigs in BOUND.values():
            for name, (res, args) in sigs.items():
                f = getattr(lib, name)
                f.restype = res
                f.argtypes = args
        return lib
    if not os.path.exists(ops.lib_path()):
        from paper_2606_18114_amd import build
        build.build(verbose=False)
    return ops.lib()


@pytest.mark.parametrize("header,count", [("tmamba_parts.h", 7), ("tmamba_decode16.h", 3)])
def test_exports_every_declared_symbol(L, header, count):
    text = open(os.path.join(ROOT, "include", header)).read()
    names = set(re.findall(r"^(?:tm_status|int64_t)\s+(tm_[a-z0-9_]+)\(", text, re.M))
    assert len(names) == count
    for n in names:
        assert hasattr(L, n), n
        assert n in BOUND[header], n


def test_scratch_sizes(L):
    for f in (L.tm_tgemm_bwd_dw_slots, lambda *a: L.tm_tgemm_bwd_dx_slots(*a, 0),
              lambda *a: L.tm_tgemm_bwd_dx_slots(*a, 1),
              lambda *a: L.tm_tgemm_fwd_scratch(*a, 128, 0),
              lambda *a: L.tm_tgemm_fwd_scratch(*a, 128, 1),
              lambda *a: L.tm_tgemm_fwd_slots(*a, 128)):
        assert f(2048, 8512, 2048) >= 0
        assert f(0, 8512, 2048) == -1
        assert f(2048, -8, 2048) == -1
        assert f(2 ** 40, 2 ** 20, 2048) == -1        # size overflow
    assert L.tm_tgemm_fwd_scratch(16, 256, 544, 128, 0) == -1
    assert L.tm_tgemm_fwd_scratch(16, 256, 512, 48, 0) == -1
    assert L.tm_tgemm_fwd_scratch(16, 256, 512, 128, 2) == -1
    assert L.tm_tgemm_fwd_slots(16, 256, 512, 48) == -1


def fwd(L, X=P, codes=P + 2 ** 24, scales=P + 2 ** 26, M=2048, N=8512, K=2048, g=128,
        Y=P + 2 ** 28, b16=0, ws=0, wsb=0, slots=0, sb=0):
    return L.tm_tgemm_fwd_parts(X, codes, scales, M, N, K, g, Y, b16, ws, wsb, slots, sb, None)


def test_tgemm_fwd_parts_validation(L):
    for kw in ("X", "codes", "scales", "Y"):
        assert fwd(L, **{kw: 0}) == EINVAL, kw
    assert fwd(L, b16=2) == EINVAL
    assert fwd(L, b16=1, ws=P + 2 ** 30, wsb=8192) == EINVAL   # the words are float32's
    assert fwd(L, M=0) == ESHAPE
    assert fwd(L, g=48) == ESHAPE
    assert fwd(L, ws=P + 2 ** 30, wsb=8191) == ESHAPE
    assert fwd(L, X=P + 2) == EALIGN
    assert fwd(L, ws=P + 2 ** 30 + 2, wsb=8192) == EALIGN
    assert fwd(L, Y=P + 4096) == EINVAL
    for b16 in (0, 1):
        big = 2 ** 28
        need = L.tm_tgemm_fwd_scratch(2048, 8512, 2048, 128, b16)
        if need > 0:
            assert fwd(L, b16=b16, slots=P + 2 ** 31, sb=need - 1) == ESHAPE
            for over in (P, P + 2 ** 24, P + 2 ** 26, P + 2 ** 28 + 16):
                assert fwd(L, b16=b16, slots=over, sb=big) == EINVAL
        assert fwd(L, b16=b16, slots=P + 2 ** 31 + 8, sb=big) == EALIGN
    if L.tm_tgemm_fwd_scratch(2048, 8512, 2048, 128, 0) > 0:
        assert fwd(L, ws=P + 2 ** 31 + 64, wsb=8192, slots=P + 2 ** 31, sb=2 ** 28) == EINVAL


def dx(L, dY=P, f32=0, b=0, codes=P + 2 ** 27, scales=P + 2 ** 28, M=2048, N=8512, K=2048, g=128,
       exact=0, dX=P + 2 ** 29, b16=0, ws=P + 2 ** 30, wsb=2 ** 28, slots=P + 2 ** 32,
       sb=2 ** 30):
    return L.tm_tgemm_bwd_dx_parts(dY, f32, b, codes, scales, M, N, K, g, exact, dX, b16, ws, wsb,
                                   slots, sb, None)


def test_tgemm_bwd_dx_parts_validation(L):
    assert L.tm_tgemm_bwd_dx_slots(2048, 8512, 2048, 0) > 0   # 64 tiles: cut
    for kw in ("dY", "codes", "scales", "dX", "ws"):
        assert dx(L, **{kw: 0}) == EINVAL, kw
    for kw in ("f32", "exact", "b16"):
        assert dx(L, **{kw: 2}) == EINVAL, kw
    assert dx(L, exact=1) == EINVAL                       # the two-pass form takes no workspace
    assert dx(L, f32=1) == EINVAL                         # no room for the rounded gradient
    assert dx(L, b=P + 2 ** 33) == EINVAL                 # nothing to round
    assert dx(L, f32=1, b=P + 2 ** 33, exact=1, ws=0) == EINVAL
    assert dx(L, N=8508) == ESHAPE
    assert dx(L, K=2112) == ESHAPE
    assert dx(L, wsb=1000) == ESHAPE
    assert dx(L, f32=1, dY=P + 8, b=P + 2 ** 33) == EALIGN
    assert dx(L, f32=1, b=P + 2 ** 33 + 8) == EALIGN
    assert dx(L, f32=1, b=P + 2 ** 20) == EINVAL          # the copy over dY
    assert dx(L, f32=1, b=P + 2 ** 29) == EINVAL          # and over dX
    assert dx(L, f32=1, b=P + 2 ** 30 + 256) == EINVAL    # and over the workspace
    assert dx(L, b16=1, slots=0, sb=0) == EINVAL          # bfloat16 sums cannot add up in place
    assert dx(L, sb=1024) == ESHAPE
    assert dx(L, slots=P + 2 ** 32 + 4) == EALIGN
    for over in (P + 64, P + 2 ** 27, P + 2 ** 28, P + 2 ** 29 + 64, P + 2 ** 30):
        assert dx(L, slots=over) == EINVAL
    assert dx(L, f32=1, b=P + 2 ** 32, slots=P + 2 ** 32) == EINVAL


def dw(L, dY=P, X=P + 2 ** 27, M=2048, N=2048, K=1024, dW=P + 2 ** 28, acc=0, slots=P + 2 ** 30,
       sb=2 ** 30):
    return L.tm_tgemm_bwd_dw_parts(dY, X, M, N, K, dW, acc, slots, sb, None)


def test_tgemm_bwd_dw_parts_validation(L):
    assert L.tm_tgemm_bwd_dw_slots(2048, 2048, 1024) > 0   # 32 tiles: cut
    for kw in ("dY", "X", "dW"):
        assert dw(L, **{kw: 0}) == EINVAL, kw
    assert dw(L, acc=2) == EINVAL
    assert dw(L, M=0) == ESHAPE
    assert dw(L, N=2044) == ESHAPE
    assert dw(L, K=1000) == ESHAPE
    assert dw(L, dW=P + 2 ** 28 + 4) == EALIGN
    assert dw(L, dW=P + 64) == EINVAL
    assert dw(L, sb=1024) == ESHAPE
    assert dw(L, slots=P + 2 ** 30 + 8) == EALIGN
    for over in (P, P + 2 ** 27 + 64, P + 2 ** 28 + 64):
        assert dw(L, slots=over) == EINVAL


def ss(L, src=P, B=16, D=2048, dst=P + 2 ** 20, part=P + 2 ** 21):
    return L.tm_rows_sumsq(src, B, D, dst, part, None)


def test_rows_sumsq_validation(L):
    for kw in ("src", "part"):
        assert ss(L, **{kw: 0}) == EINVAL, kw
    assert ss(L, B=0) == ESHAPE
    assert ss(L, B=65536) == ESHAPE
    assert ss(L, D=0) == ESHAPE
    for kw in ("src", "dst", "part"):
        assert ss(L, **{kw: P + 2 ** 22 + 2}) == EALIGN, kw
    assert ss(L, dst=P) == EINVAL
    assert ss(L, part=P + 64) == EINVAL
    assert ss(L, part=P + 2 ** 20 + 64) == EINVAL


def r16(L, src=P, part=P + 2 ** 20, nparts=64, nw=P + 2 ** 21, eps=1e-5, codes=P + 2 ** 22,
        s16=P + 2 ** 25, B=16, N=8512, K=2048, g=128, y=P + 2 ** 26, acc=0, po=P + 2 ** 28,
        adv=P + 2 ** 29):
    return L.tm_tgemv_rms16(src, part, nparts, nw, eps, codes, s16, B, N, K, g, y, acc, po, adv,
                            None)


def test_tgemv_rms16_validation(L):
    for kw in ("src", "nw", "codes", "s16", "y"):
        assert r16(L, **{kw: 0}) == EINVAL, kw
    assert r16(L, eps=-1.0) == EINVAL
    assert r16(L, eps=float("nan")) == EINVAL
    assert r16(L, acc=2) == EINVAL
    assert r16(L, B=0) == ESHAPE
    assert r16(L, B=17) == ESHAPE
    assert r16(L, N=0) == ESHAPE
    assert r16(L, nparts=0) == ESHAPE
    assert r16(L, part=0) == ESHAPE                       # nparts without part
    assert r16(L, g=32) == ESHAPE
    assert r16(L, g=512) == ESHAPE
    assert r16(L, K=4224) == ESHAPE                       # x of 16 rows is past the LDS
    assert r16(L, K=2112) == ESHAPE
    assert r16(L, src=P + 4) == EALIGN
    assert r16(L, nw=P + 2 ** 21 + 8) == EALIGN
    assert r16(L, codes=P + 2 ** 22 + 4) == EALIGN
    assert r16(L, s16=P + 2 ** 25 + 1) == EALIGN
    for kw in ("part", "y", "po", "adv"):
        assert r16(L, **{kw: P + 2 ** 30 + 2}) == EALIGN, kw
    for kw in ("y", "po", "adv"):                         # outputs over inputs and each other
        for over in (P, P + 2 ** 20, P + 2 ** 21, P + 2 ** 22, P + 2 ** 25):
            assert r16(L, **{kw: over}) == EINVAL, (kw, over - P)
    assert r16(L, po=P + 2 ** 26 + 64) == EINVAL
    assert r16(L, adv=P + 2 ** 26) == EINVAL
    assert r16(L, adv=P + 2 ** 28) == EINVAL


def mgp(L, z=P, B=1, H=64, hd=64, ds=128, cs=P + 2 ** 20, pos=P + 2 ** 21, ss=P + 2 ** 22,
        cw=P + 2 ** 24, cb=P + 2 ** 25, dtb=P + 2 ** 26, al=P + 2 ** 26 + 4096,
        D=P + 2 ** 26 + 8192, gated=P + 2 ** 28, part=P + 2 ** 29):
    return L.tm_mixer_gate_part(z, B, H, hd, ds, cs, pos, ss, cw, cb, dtb, al, D, gated, part,
                                None)


def test_mixer_gate_part_validation(L):
    for kw in ("z", "cs", "pos", "ss", "cw", "cb", "dtb", "al", "D", "gated", "part"):
        assert mgp(L, **{kw: 0}) == EINVAL, kw
    assert mgp(L, B=0) == ESHAPE
    assert mgp(L, hd=128) == ESHAPE
    assert mgp(L, gated=P + 2 ** 28 + 2) == EALIGN
    assert mgp(L, part=P + 2 ** 29 + 2) == EALIGN
    assert mgp(L, gated=P + 2 ** 22 + 64) == EINVAL
    # the partial sums over every other operand
    for over in (P, P + 2 ** 20, P + 2 ** 21, P + 2 ** 22, P + 2 ** 24, P + 2 ** 25, P + 2 ** 26,
                 P + 2 ** 26 + 4096, P + 2 ** 26 + 8192, P + 2 ** 28):
        assert mgp(L, part=over) == EINVAL, hex(over - P)
