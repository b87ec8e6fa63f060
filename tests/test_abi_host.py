"""Host-side checks of the C ABI that need no GPU: the library builds and loads, exports
every symbol the header declares, and rejects bad arguments before launching anything."""
import ctypes
import math
import os
import re

import pytest

from paper_2502_13542_amd import binding as B
from paper_2502_13542_amd.synth import LayerShape

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLAMA = LayerShape(32, 8, 128, 128, 4, 128, 512, "bf16")


@pytest.fixture(scope="module")
def lib():
    return B.load_library()


def test_exports_every_declared_symbol(lib):
    text = open(os.path.join(ROOT, "include", "actqkv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(actqkv_[a-z_]+)\s*\(", text))
    assert {"actqkv_build_probe", "actqkv_score_blocks", "actqkv_select",
            "actqkv_retrieval_attention"} <= declared
    for name in declared:
        assert hasattr(lib, name), f"{name} is declared in actqkv.h but not exported"
    assert declared == set(B.SIGNATURES), "binding and header disagree"
    assert lib.actqkv_version() == int(re.search(r"#define ACTQKV_VERSION (\d+)", text).group(1))


def test_header_is_plain_c(tmp_path):
    """include/actqkv.h compiles as C99 with warnings on (no C++ or HIP types in the signatures)."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no gcc")
    src = tmp_path / "use_header.c"
    src.write_text('#include "actqkv.h"\nint use(void) { return actqkv_version() > 0 ? ACTQKV_OK : ACTQKV_EINVAL; }\n')
    res = subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I", os.path.join(ROOT, "include"),
                          "-c", str(src), "-o", str(tmp_path / "use_header.o")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr


def test_struct_layout_matches_header():
    assert ctypes.sizeof(B.CShape) == 40
    assert B.CShape.softmax_scale.offset == 32 and B.CShape.var_eps.offset == 36


def test_sizes(lib):
    cs = B.c_shape(LLAMA)
    assert B.stats_floats(cs) == 4 + 2 * 4096
    ws = B.workspace_bytes(cs, 1, 512, 1024, 32)
    assert ws >= 4096 and ws % 256 == 0
    assert B.workspace_bytes(cs, 16, 1, 520, 32) >= 4096


A16 = 0x10000  # fake, aligned, never dereferenced: every check below fails before a launch


def _probe(lib, cs, **kw):
    a = dict(batch=1, m=512, q=A16, stats=A16, upd=1, probe=A16, pkv=A16, pn=A16, w=None, ws=A16,
             wsb=1 << 30)
    a.update(kw)
    return lib.actqkv_build_probe(ctypes.byref(cs), a["batch"], a["m"], a["q"], a["stats"], a["upd"],
                                  a["probe"], a["pkv"], a["pn"], a["w"], a["ws"], a["wsb"], None)


def test_workspace_serves_smaller_calls(lib):
    """A workspace sized for (batch, m) is at least what any call with fewer entries or shorter
    windows asks for: few short windows need partial results, many long ones none, and a
    window too long for the matrix-core kernel needs no attention scratch at all."""
    for sh in (LLAMA, LayerShape(8, 2, 128, 128, 4, 128, 256, "bf16"), LayerShape(8, 2, 64, 128, 4, 128, 256, "fp32")):
        cs = B.c_shape(sh)
        for batch, m in ((32, 512), (1, 4096), (4, 2048), (16, 1)):
            big = B.workspace_bytes(cs, batch, m, 1024, 32)
            for b2 in sorted(b for b in {1, 2, batch // 2 or 1, batch} if b <= batch):
                for m2 in sorted(x for x in {1, 77, 128, m // 2 or 1, m} if x <= m):
                    assert B.workspace_bytes(cs, b2, m2, 1024, 32) <= big, (sh, batch, m, b2, m2)


def _cut_us(cut, hk, batch, m, k_cap, cus):
    """The figures by which the attention of several windows is cut up: microseconds of the busiest compute unit."""
    rows, tiles, slots = cut[:3]
    tile, merge, piece = {256: (3.7, 6.0, 1.1), 128: (2.1, 3.5, 0.7), 64: (1.5, 2.0, 0.5)}[rows]
    longest, pieces, rounds = (128 + 512 + m) / 128 + k_cap / 2, slots // tiles, batch * hk * slots / cus
    us = max(math.ceil(longest / pieces), rounds * (longest - m / 256) / pieces) * tile + 8 * max(rounds, 1.0)
    return us + (merge + piece * pieces if slots > tiles else 0.0)


def _best_cut(hq, hk, batch, m, k_cap, cus):
    cuts = []
    for ks in (1, 2, 4):
        tiles = -(-m * (hq // hk) * ks // 256)
        room = max(cus // (batch * hk), tiles)
        pieces = min(room // tiles, 8)
        cuts.append((256 // ks, tiles, pieces * tiles + (room - pieces * tiles if ks == 1 and pieces < 8 else 0)))
    return min(cuts, key=lambda c: _cut_us(c, hk, batch, m, k_cap, cus))


@pytest.mark.parametrize("hq,hk,cus", [(32, 8, 256), (28, 4, 256), (8, 2, 256), (32, 32, 256), (8, 8, 224), (28, 4, 224)])
def test_cut_of_a_window_with_one_term_probabilities(lib, hq, hk, cus):
    """Windows of bf16 probabilities of one term: they are rounded against the maximum of the wavefronts that share a tile, so
    the output's bits belong to the cut, and the cut is the least by one set of figures, whether a window comes alone or not."""
    cs = B.c_shape(LayerShape(hq, hk, 128, 128, 4, 128, 512, "bf16"))
    for batch in (1, 5):
        for k_cap in (6, 16, 32):
            for m in list(range(2, 1100, 37)) + [512, 513, 640, 678, 700, 1024, 2441, 2500]:
                assert B.prefill_cut(cs, batch, m, k_cap, cus)[:3] == _best_cut(hq, hk, batch, m, k_cap, cus), (batch, k_cap, m)
    for bad in (dict(batch=0), dict(m=1), dict(m=8193), dict(k_cap=65), dict(cus=257)):
        with pytest.raises(B.ActQKVError):
            B.prefill_cut(cs, **{**dict(batch=1, m=512, k_cap=8, cus=256), **bad})


@pytest.mark.parametrize("hq,hk", [(32, 8), (8, 2), (32, 32)])
def test_cut_of_a_window_with_64_channels(lib, hq, hk):
    """Another cut for a single window is one by which four of them in a call, which take the same, are priced no higher."""
    cs = B.c_shape(LayerShape(hq, hk, 64, 128, 4, 128, 512, "bf16"))
    others = 0
    for k_cap in (6, 16, 32):
        for m in list(range(2, 4096, 61)) + [640, 768, 1200]:
            cut, plain = B.prefill_cut(cs, 1, m, k_cap)[:3], _best_cut(hq, hk, 1, m, k_cap, 256)
            others += cut != plain
            assert cut == plain or _cut_us(cut, hk, 4, m, k_cap, 256) <= _cut_us(plain, hk, 4, m, k_cap, 256), (k_cap, m)
    assert others > 0


def test_build_probe_rejects(lib):
    cs = B.c_shape(LLAMA)
    assert _probe(lib, cs, batch=0) == -1
    assert _probe(lib, cs, m=0) == -1
    assert _probe(lib, cs, q=None) == -1 and b"q_win" in lib.actqkv_last_error()
    assert _probe(lib, cs, q=A16 + 4) == -3
    assert _probe(lib, cs, ws=None) == -4
    assert _probe(lib, cs, wsb=100) == -4 and b"needs" in lib.actqkv_last_error()
    assert lib.actqkv_build_probe(None, 1, 1, A16, A16, 0, A16, A16, A16, None, A16, 1 << 20, None) == -1
    # consecutive windows of one sequence: need the update bit and m >= 2; unknown bits
    assert _probe(lib, cs, batch=4, upd=B.PROBE_WINDOW_CHAIN) == -1 and b"ACTQKV_STATS_UPDATE" in lib.actqkv_last_error()
    assert _probe(lib, cs, batch=4, m=1, upd=B.PROBE_WINDOW_CHAIN | B.STATS_UPDATE) == -1
    assert _probe(lib, cs, upd=8) == -1 and b"unknown bits" in lib.actqkv_last_error()


def test_window_step_rejects(lib):
    """What one of the four calls refuses, before anything is launched."""
    cs = B.c_shape(LLAMA)
    base = dict(shape=ctypes.byref(cs), batch=1, m=512, q=A16, stats=A16, upd=1, probe=A16, pkv=A16, pn=A16, w=None, rep=A16,
                rs=0, nbs=400, nbb=1, nbe=A16, sc=A16, ss=512, k=32, fl=0, bud=None, rest=None, idx=A16, ns=A16, th=None, b=None,
                kc=A16, vc=A16, cst=0, nb=512, n_ctx=A16, out=A16, lse=None, ws=A16, wsb=1 << 30, stream=None)
    call = lambda **kw: lib.actqkv_window_step(*{**base, **kw}.values())  # noqa: E731
    assert call(shape=None) == -1
    assert call(q=None) == -1 and b"q_win" in lib.actqkv_last_error()
    assert call(rep=A16 + 4) == -3 and b"rep_keys" in lib.actqkv_last_error()
    assert call(ss=100) == -1 and b"score_stride" in lib.actqkv_last_error()
    assert call(k=65) == -2 and call(idx=None) == -1
    assert call(bud=A16) == -1 and b"together" in lib.actqkv_last_error()
    assert call(kc=None) == -1 and b"k_cache" in lib.actqkv_last_error()
    assert call(nb=3) == -1 and b"cannot hold" in lib.actqkv_last_error()
    assert call(wsb=100) == -4


def test_decode_step_rejects(lib):
    """What one of the two calls refuses, before anything is launched."""
    cs = B.c_shape(LLAMA)
    base = dict(shape=ctypes.byref(cs), batch=2, q=A16, kn=A16, vn=A16, pos=A16, kc=A16, vc=A16, cst=1 << 30, rep=A16, rs=1 << 24,
                nbs=64, nbb=1, nbe=A16, probe=None, pkv=None, pn=None, sc=A16, ss=64, k=32, fl=0, bud=None, rest=None, idx=A16,
                ns=A16, th=None, b=None, nb=64, n_ctx=A16, out=A16, lse=None, ws=A16, wsb=1 << 30, stream=None)
    call = lambda **kw: lib.actqkv_decode_step(*{**base, **kw}.values())  # noqa: E731
    assert call(shape=None) == -1 and call(q=None) == -1 and call(kn=None) == -1 and call(rep=A16 + 4) == -3
    assert call(ss=10) == -1 and call(k=65) == -2 and call(idx=None) == -1 and call(bud=A16) == -1
    assert call(fl=B.DECODE_SCORES_ONLY) == -1 and call(fl=B.SELECT_GIVEN_COUNT) == -1
    assert call(out=None) == -1 and call(n_ctx=None) == -1 and call(kc=None) == -1
    assert call(kn=None, vn=None, pos=None, kc=None) == -1 and b"k_cache" in lib.actqkv_last_error()
    assert call(wsb=100) == -4 and call(ws=None) == -4


@pytest.mark.parametrize("field,value,code", [("head_dim", 96, -2), ("n_kv_heads", 5, -2),
                                              ("block_size", 64, -2), ("n_rep", 17, -2),
                                              ("n_init", 100, -2), ("dtype", 7, -1),
                                              ("n_q_heads", 0, -1), ("softmax_scale", -1.0, -1)])
def test_shape_rejects(lib, field, value, code):
    cs = B.c_shape(LLAMA)
    setattr(cs, field, value)
    assert _probe(lib, cs) == code
    assert B.stats_floats(cs) == 0


def test_score_select_attention_reject(lib):
    cs = B.c_shape(LLAMA)
    sb = lambda **k: lib.actqkv_score_blocks(ctypes.byref(cs), k.get("batch", 1), A16, A16,
                                             k.get("rep", A16), k.get("stride", 0), k.get("cap", 64), 1,
                                             A16, A16, k.get("ss", 64), None)
    assert sb(rep=None) == -1 and sb(rep=A16 + 8) == -3 and sb(ss=10) == -1 and sb(cap=-1) == -1
    assert sb(batch=2, stride=8) == -1 and sb(stride=4) == -3 and sb(cap=9000, ss=9000) == -2
    se = lambda **k: lib.actqkv_select(1, A16, 64, 64, 1, A16, k.get("k_cap", 32), k.get("flags", 0),
                                       k.get("bud"), k.get("rest"), k.get("idx", A16), A16, None, None, None)
    assert se(k_cap=0) == -2 and se(k_cap=65) == -2 and se(idx=None) == -1 and se(flags=2) == -1
    assert se(bud=A16 + 2, rest=A16) == -3 and se(bud=A16) == -1 and se(rest=A16) == -1
    at = lambda **k: lib.actqkv_retrieval_attention(ctypes.byref(cs), 1, k.get("m", 512), A16,
                                                    k.get("kc", A16), A16, 0, k.get("cap", 64), A16, A16,
                                                    A16, 32, k.get("out", A16), None, k.get("ws", A16),
                                                    k.get("wsb", 1 << 30), None)
    assert at(kc=None) == -1 and at(out=A16 + 2) == -3 and at(ws=None) == -4 and at(wsb=8) == -4
    assert at(m=0) == -1 and at(cap=2) == -1 and at(cap=0) == -1
    sp = lambda **k: lib.actqkv_score_blocks_per_head(ctypes.byref(cs), 1, k.get("probe", A16), k.get("rep", A16), 0,
                                                      k.get("cap", 64), 1, A16, A16, k.get("ss", 64), None)
    assert sp(probe=None) == -1 and sp(rep=A16 + 8) == -3 and sp(ss=10) == -1 and sp(cap=9000, ss=9000) == -2
    assert lib.actqkv_retrieval_attention_per_head(ctypes.byref(cs), 1, 512, A16, None, A16, 0, 64, A16, A16, A16, 32,
                                                   A16, None, A16, 1 << 30, None) == -1
    ap = lambda **k: lib.actqkv_append_kv_probe(ctypes.byref(cs), 1, k.get("q", A16), A16, A16, A16, A16, A16, 0, None,
                                                0, k.get("cap", 64), k.get("probe", A16), A16, A16, None)
    assert ap(q=None) == -1 and b"q_tok" in lib.actqkv_last_error() and ap(probe=None) == -1
    assert ap(cap=0) == -1 and ap(q=A16 + 2) == -3
    ga = lambda **k: lib.actqkv_gather_blocks(ctypes.byref(cs), 1, k.get("ks", A16), A16, 0, k.get("nbs", 64), A16,
                                              A16, k.get("k_cap", 32), k.get("kc", A16), A16, 0, k.get("cap", 64),
                                              k.get("slot0", 1), None, None)
    assert ga(ks=None) == -1 and ga(kc=A16 + 4) == -3 and ga(k_cap=65) == -2 and ga(nbs=0) == -1
    assert ga(slot0=40) == -1 and b"outside the cache" in lib.actqkv_last_error() and ga(slot0=-1) == -1
    with pytest.raises(B.ActQKVError):
        B._check(at(wsb=8))


def test_workspace_serves_every_launch_shape(lib):
    """The launch shape is an argument of the attention call, not process-wide state: a workspace
    of actqkv_workspace_bytes is accepted with every first_cus (the host checks run up to the
    launch, which fails without a GPU: any code but EWORKSPACE and the argument errors)."""
    cs = B.c_shape(LLAMA)
    for batch, m in ((1, 512), (2, 512), (32, 512), (1, 96)):
        full = B.workspace_bytes(cs, batch, m, 1024, 32)
        for cus in (1, 8, 64, 192, 224, 256):
            rc = lib.actqkv_retrieval_attention_teams(
                ctypes.byref(cs), batch, m, A16, A16, A16, 0, 1024, A16, A16, A16, 32, A16, None, A16, full,
                cus, 0, None, None)
            assert rc in (0, -5), (batch, m, cus, B.last_error())


def test_attention_cache_larger_than_a_selection(lib):
    """The attention selects nothing, so the 8192-block limit of one selection does not apply to
    its cache; the calls that select keep it."""
    cs = B.c_shape(LLAMA)
    att = lambda nb: lib.actqkv_retrieval_attention(
        ctypes.byref(cs), 1, 512, A16, A16, A16, 0, nb, A16, A16, A16, 32, A16, None, A16, 1 << 30, None)
    assert att(8193) in (0, -5) and att(1 << 20) in (0, -5)
    assert att((1 << 23) + 1) == -2 and b"2^30" in lib.actqkv_last_error()
    sel = lambda nb: lib.actqkv_select(1, A16, nb, nb, 0, A16, 32, 0, None, None, A16, A16, None, None, None)
    assert sel(8193) == -2 and b"8192" in lib.actqkv_last_error()


def test_copy_bytes_rejects(lib):
    assert lib.actqkv_copy_bytes(None, A16, 1024, None) == -1
    assert lib.actqkv_copy_bytes(A16, None, 1024, None) == -1
    assert lib.actqkv_copy_bytes(A16, A16 + 4096, 1000, None) == -1      # not a multiple of 16
    assert lib.actqkv_copy_bytes(A16 + 4, A16 + 4096, 1024, None) == -3  # alignment
    assert lib.actqkv_copy_bytes(A16, A16 + 4096, 0, None) == 0          # nothing to do, nothing launched


def test_append_kv_rejects(lib):
    cs = B.c_shape(LLAMA)
    call = lambda **kw: lib.actqkv_append_kv(ctypes.byref(cs), kw.get("batch", 1), kw.get("m", 512),
                                             kw.get("k", A16), kw.get("v", A16), kw.get("pos0", A16),
                                             kw.get("kc", A16), kw.get("vc", A16), kw.get("cs", 0),
                                             kw.get("rep", A16), kw.get("rs", 0), kw.get("nb", 8), None)
    assert call(m=0) == -1 and call(batch=0) == -1 and call(nb=0) == -1
    assert call(k=None) == -1 and call(pos0=None) == -1 and call(vc=None) == -1
    assert call(k=A16 + 2) == -3 and call(cs=12) == -3
    assert call(batch=2, cs=8) == -1                       # stride smaller than one sequence's cache


def test_decode_retrieve_rejects(lib):
    cs = B.c_shape(LLAMA)
    call = lambda **k: lib.actqkv_decode_retrieve(
        ctypes.byref(cs), k.get("batch", 1), k.get("q", A16), k.get("kn", A16), k.get("vn", A16),
        k.get("pos0", A16), k.get("kc", A16), A16, k.get("cs", 0), k.get("rep", A16), k.get("rs", 0),
        k.get("cap", 64), 1, k.get("nb_end", A16), None, None, None, k.get("scores", A16), k.get("ss", 64),
        k.get("k_cap", 32), k.get("flags", 0), k.get("bud"), k.get("rest"), k.get("idx", A16), A16, None, None, None)
    assert call(q=None) == -1 and b"q_tok" in lib.actqkv_last_error() and call(q=A16 + 2) == -3
    assert call(kn=None) == -1 and call(pos0=None) == -1 and call(kc=None) == -1     # a partial cache update
    assert call(rep=None) == -1 and call(nb_end=None) == -1 and call(scores=None) == -1 and call(idx=None) == -1
    assert call(cap=0) == -1 and call(cap=9000, ss=9000) == -2 and call(ss=10) == -1
    assert call(k_cap=0) == -2 and call(k_cap=65) == -2 and call(flags=4) == -1
    assert call(bud=A16) == -1 and call(bud=A16 + 2, rest=A16) == -3
    assert call(batch=2, cs=8) == -1 and call(batch=2, cs=1 << 40, rs=8) == -1 and call(cs=12) == -3


def test_decode_select_attention_rejects(lib):
    cs = B.c_shape(LLAMA)
    call = lambda **k: lib.actqkv_decode_select_attention(
        ctypes.byref(k.get("shape", cs)), k.get("batch", 1), k.get("q", A16), k.get("kc", A16), A16, k.get("stride", 0),
        k.get("cap", 64), k.get("n_ctx", A16), k.get("scores", A16), k.get("ss", 64), 1, k.get("nb_end", A16),
        k.get("k_cap", 32), k.get("flags", 0), k.get("bud"), k.get("rest"), k.get("after"), k.get("idx", A16),
        k.get("n_sel", A16), None, None, k.get("out", A16), None, k.get("ws", A16), k.get("wsb", 1 << 30), None)
    assert call(q=None) == -1 and call(kc=A16 + 2) == -3 and call(scores=None) == -1 and call(out=None) == -1
    assert call(idx=None) == -1 and call(n_sel=None) == -1 and call(n_ctx=None) == -1 and call(nb_end=None) == -1
    assert call(cap=0) == -1 and call(ss=10) == -1 and call(k_cap=65) == -2 and call(flags=2) == -1
    assert call(bud=A16) == -1 and call(bud=A16, rest=A16, after=A16) == -1     # in place is not allowed
    assert b"budget_after" in lib.actqkv_last_error()
    assert call(batch=2, stride=8) == -1 and call(stride=4) == -3
    assert call(ws=None) == -4 and call(wsb=8) == -4
    fp32 = B.c_shape(LayerShape(8, 2, 64, 128, 4, 128, 256, "fp32"))
    assert call(shape=fp32) == -2                                               # a bf16, head_dim 128 kernel


def test_decode_layer_rejects(lib):
    """The whole decode layer in one launch: everything is refused on the host before a kernel runs."""
    cs = B.c_shape(LLAMA)
    call = lambda **k: lib.actqkv_decode_layer(
        ctypes.byref(k.get("shape", cs)), k.get("batch", 1), k.get("q", A16), k.get("kn", A16), k.get("vn", A16),
        k.get("kc", A16), A16, k.get("cs", 0), k.get("rep", A16), k.get("rs", 0), k.get("cap", 64),
        k.get("n_ctx", A16), 1, k.get("nb_end", A16), k.get("scores", A16), k.get("ss", 64), k.get("k_cap", 32),
        k.get("flags", 0), k.get("bud"), k.get("rest"), k.get("after"), k.get("idx", A16), k.get("n_sel", A16),
        None, None, k.get("out", A16), None, k.get("ws", A16), k.get("wsb", 1 << 30), None)
    assert call(q=None) == -1 and call(kn=None) == -1 and b"together" in lib.actqkv_last_error()
    assert call(kc=None) == -1 and call(rep=None) == -1 and call(kc=A16 + 2) == -3
    assert call(n_ctx=None) == -1 and call(nb_end=None) == -1 and call(scores=None) == -1
    assert call(idx=None) == -1 and call(n_sel=None) == -1 and call(out=None) == -1
    assert call(cap=0) == -1 and call(cap=9000, ss=9000) == -2 and call(ss=10) == -1
    assert call(k_cap=0) == -2 and call(k_cap=65) == -2
    assert call(flags=2) == -1 and call(flags=8) == -1 and b"unknown flag" in lib.actqkv_last_error()
    assert call(bud=A16) == -1 and call(bud=A16, rest=A16, after=A16) == -1
    assert b"budget_after" in lib.actqkv_last_error()
    assert call(batch=385) == -2 and b"batch" in lib.actqkv_last_error()
    assert call(batch=2, cs=8) == -1 and call(batch=2, cs=1 << 40, rs=8) == -1 and call(cs=12) == -3
    assert call(ws=None) == -4 and call(wsb=8) == -4
    fp32 = B.c_shape(LayerShape(8, 2, 64, 128, 4, 128, 256, "fp32"))
    assert call(shape=fp32) == -2


def test_blocked_representatives_equal_the_token_major_rule():
    """The harness rule for the representative keys of a synthetic cache, on a blocked cache and on
    token-major keys: the same keys (it is an input recipe; the oracle's rule is pinned on its own)."""
    import torch
    from paper_2502_13542_amd import synth
    g = torch.Generator().manual_seed(5)
    k = torch.randn(3 * 128, 2, 16, generator=g)
    k[130] = k[131]                                       # a tie: the earlier position wins
    blocked = k.reshape(3, 128, 2, 16).permute(0, 2, 1, 3)[None].contiguous()
    assert torch.equal(synth.pick_rep_keys(k, 128, 4), synth.pick_rep_keys_blocked(blocked, 4)[0])


def test_retrieval_attention_teams_rejects(lib):
    cs = B.c_shape(LLAMA)
    call = lambda **k: lib.actqkv_retrieval_attention_teams(
        ctypes.byref(cs), 32, 512, k.get("q", A16), A16, A16, 0, 1024, A16, A16, A16, 32, k.get("out", A16), None,
        k.get("ws", A16), k.get("wsb", 1 << 30), k.get("first_cus", 224), k.get("late_cus", 32), None, None)
    assert call(late_cus=4) == -1 and call(late_cus=300) == -1 and call(late_cus=-1) == -1
    assert b"late_cus" in lib.actqkv_last_error()
    assert call(first_cus=0) == -1 and call(first_cus=257) == -1 and b"first_cus" in lib.actqkv_last_error()
    assert call(q=None) == -1 and call(out=A16 + 2) == -3 and call(ws=None) == -4 and call(wsb=8) == -4


def test_retrieval_attention_windows_rejects(lib):
    cs, fp32 = B.c_shape(LLAMA), B.c_shape(LayerShape(32, 8, 128, 128, 4, 128, 512, "fp32"))
    call = lambda shape=cs, nw=4, m=512, **k: lib.actqkv_retrieval_attention_windows(
        ctypes.byref(shape), nw, m, k.get("q", A16), A16, A16, k.get("nb", 64), A16, A16, A16, k.get("k_cap", 16),
        k.get("out", A16), k.get("lse"), k.get("ws", A16), k.get("wsb", 1 << 30), k.get("cus", 224), None)
    assert call(cus=0) == -1 and call(cus=257) == -1 and b"cus" in lib.actqkv_last_error()
    assert call(nw=0) == -1 and call(nw=1025) == -2 and call(m=0) == -1 and call(m=8193) == -2
    assert call(shape=fp32) == -2 and call(m=1) == -2 and b"bf16" in lib.actqkv_last_error()
    assert call(nb=3) == -1 and call(k_cap=65) == -2
    assert call(q=None) == -1 and call(out=A16 + 2) == -3 and call(lse=A16 + 2) == -3
    one = lib.actqkv_workspace_bytes(ctypes.byref(cs), 1, 512, 64, 16)
    assert call(ws=None) == -4 and call(nw=200, wsb=one) == -4 and b"needs" in lib.actqkv_last_error()


def test_gather_blocks_cached_rejects(lib):
    cs = B.c_shape(LLAMA)
    call = lambda nw=4, k_cap=16, **k: lib.actqkv_gather_blocks_cached(
        ctypes.byref(cs), nw, k.get("store", A16), A16, k.get("nb_store", 256), k.get("idx", A16), A16, k_cap,
        k.get("cache", A16), A16, k.get("nb", 300), k.get("slot0", 1), k.get("n_slots", 128), *k.get("here0", (0, 0, 0)),
        *k.get("here1", (0, 0, 0)), k.get("group", 0), k.get("state", A16), A16, None)
    assert call(k_cap=0) == -2 and call(k_cap=65) == -2 and call(nw=0) == -2 and call(nw=17) == -2
    assert b"selections" in lib.actqkv_last_error()
    assert call(nb_store=0) == -1 and call(n_slots=127) == -1 and call(n_slots=513) == -1
    assert call(slot0=-1) == -1 and call(slot0=173) == -1 and b"outside the cache" in lib.actqkv_last_error()
    assert call(group=-1) == -1
    # a range that lies in the cache may not touch the slots (1 .. 128) nor leave the cache
    for here in ((0, 2, 0), (5, 7, 128), (0, 8, 293), (-1, 3, 200), (0, 3, -1)):
        assert call(here0=here) == -1 and call(here1=here) == -1, here
        assert b"overlap the slots" in lib.actqkv_last_error()
    assert call(store=None) == -1 and call(cache=A16 + 2) == -3 and call(idx=A16 + 2) == -3 and call(state=None) == -1


def test_retrieval_attention_static_rejects(lib):
    """The entry point that allocates nothing: argument errors as in actqkv_retrieval_attention, and
    a call whose scratch need exceeds the library's own array is refused before anything runs."""
    cs = B.c_shape(LLAMA)
    call = lambda shape=cs, batch=1, m=512, **k: lib.actqkv_retrieval_attention_static(
        ctypes.byref(shape), batch, m, k.get("q", A16), A16, A16, 0, k.get("nb", 1024), A16, A16, A16,
        k.get("k_cap", 32), k.get("out", A16), None, None)
    assert call(q=None) == -1 and call(out=A16 + 2) == -3 and call(k_cap=65) == -2 and call(m=0) == -1
    big = B.c_shape(LayerShape(128, 16, 128, 128, 4, 128, 512, "bf16"))
    assert call(shape=big, batch=1024, m=1, nb=2) == -4
    msg = lib.actqkv_last_error().decode()
    assert "scratch" in msg and str(32 << 20) in msg
    # the largest batches of the other kinds have a workgroup per (sequence, KV head) and need no partial results
    for shape in (LayerShape(64, 64, 128, 128, 4, 128, 256, "fp32"), LayerShape(256, 64, 64, 128, 4, 128, 256, "bf16"),
                  LayerShape(256, 256, 64, 128, 4, 128, 256, "fp32")):
        assert call(shape=B.c_shape(shape), batch=1024, m=1, nb=2) in (0, -5), lib.actqkv_last_error()


def test_cutoff_budgets_and_select_modes_reject(lib):
    f = ctypes.c_float
    call = lambda batch=2, L=32, k=8.0, cap=32, th=A16, b=A16, c=A16, left=None: \
        lib.actqkv_cutoff_budgets(batch, L, f(k), cap, th, b, c, left, None)
    assert call(batch=0) == -1 and call(k=0.0) == -1 and call(L=0) == -2 and call(L=2000) == -2
    assert call(cap=0) == -2 and call(cap=65) == -2
    assert call(th=None) == -1 and call(b=None) == -1 and call(c=A16 + 2) == -3 and call(left=A16 + 1) == -3
    sel = lambda flags, theta=A16, bud=None, rest=None: lib.actqkv_select(
        1, A16, 64, 64, 0, A16, 8, flags, bud, rest, A16, A16, theta, None, None)
    assert sel(B.SELECT_DENSITY_ONLY | B.SELECT_GIVEN_COUNT) == -1 and b"exclude" in lib.actqkv_last_error()
    assert sel(B.SELECT_DENSITY_ONLY, theta=None) == -1 and b"theta" in lib.actqkv_last_error()
    assert sel(B.SELECT_GIVEN_COUNT, bud=A16, rest=A16) == -1 and b"cut-off state" in lib.actqkv_last_error()
    assert sel(32) == -1 and b"unknown flag" in lib.actqkv_last_error()


def test_cutoff_next_step_rejects(lib):
    f = ctypes.c_float
    call = lambda batch=2, L=32, k=8.0, prior=6.0, prev=A16, ts=A16, ns=A16, b=A16, r=A16: \
        lib.actqkv_cutoff_next_step(batch, L, f(k), f(prior), prev, ts, ns, b, r, None)
    assert call(batch=0) == -1 and call(k=0.0) == -1 and call(prior=-1.0) == -1
    assert call(L=0) == -2 and call(L=2000) == -2
    assert call(ts=None) == -1 and call(b=None) == -1 and call(r=A16 + 2) == -3


def test_another_build_may_lack_entry_points(tmp_path):
    """ACTQKV_LIB names another build for comparisons, an older one too: what it lacks raises when it is called."""
    import subprocess
    import sys
    (tmp_path / "old.c").write_text("int actqkv_version(void) { return 1; }\n"
                                    "const char* actqkv_last_error(void) { return \"\"; }\n")
    old = str(tmp_path / "old.so")
    subprocess.run(["gcc", "-shared", "-fPIC", str(tmp_path / "old.c"), "-o", old], check=True)
    code = """
from paper_2502_13542_amd import binding as B
print(B.version())
try:
    B.select(1, None, 1, 1, 0, None, 1, None, None, None, None)
except RuntimeError as e:
    print("lacks" if "does not have this entry point" in str(e) else e)
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120,
                       env={**os.environ, "ACTQKV_LIB": old})
    assert r.returncode == 0 and r.stdout.split() == ["1", "lacks"], r.stdout + r.stderr[-1000:]


def test_pinned_verdict_does_not_outlive_its_tensor(monkeypatch):
    """A host tensor at an address where a pinned one was before is asked about anew (and the other way round): a
    kernel that reads pageable memory in place faults."""
    import torch
    memory, verdict = bytearray(64), [True]
    monkeypatch.setattr(torch.Tensor, "is_pinned", lambda self, *a: verdict[0])
    at = lambda: torch.frombuffer(memory, dtype=torch.uint8)
    assert B._ptr_readable(at()) == at().data_ptr()
    verdict[0] = False
    with pytest.raises(B.ActQKVError, match="pinned"):
        B._ptr_readable(at())
    verdict[0] = True
    assert B._ptr_readable(at()) == at().data_ptr()


def test_cpp_exceptions_reach_python():
    """What torch throws while a call's arguments are taken (no GPU for the current stream, a tensor
    without memory) is a Python exception, not the end of the process."""
    import subprocess
    import sys
    code = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2502_13542_amd import binding as B
def call(t):
    try:
        B.cutoff_next_step(1, 1, 1., 1., t, t, t, t, t)
    except RuntimeError:
        print("raised")
    return t
call(None)
with FakeTensorMode():
    torch.func.vmap(call)(torch.empty(4, 64, device="cuda"))
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-1000:]
    assert r.stdout.split() == ["raised", "raised"]


@pytest.mark.parametrize("lead", [(), (2,)])
def test_a_window_scores_no_blocks_that_its_keys_do_not_hold(monkeypatch, lead):
    """The scoring of a window may read every block that it is told of: of a loose bound of the eligible ones, those
    that rep_keys holds."""
    import torch
    from paper_2502_13542_amd import harness as H
    sh = LayerShape(8, 2, 64, 128, 4, 128, 256, "fp32")
    runner = H.LayerRunner(sh, 2 if lead else 1, 16, 40, 4, "cpu")
    told = []
    monkeypatch.setattr(H.B, "window_step", lambda *a, **k: told.append(a[12]))
    cache = torch.zeros(*lead, 1)
    for held, bound in ((9, 40), (9, 5), (40, 100), (0, 3)):
        runner.step(cache, cache, cache, torch.zeros(*lead, held, 4, 2, 64), None, None, bound, None)
    assert told == [9, 5, 40, 1]


def test_overlapped_host_cache_pass_refuses_capture(monkeypatch):
    """Under capture nothing is enqueued: the end of a capture of its streams crashes the process."""
    import torch
    from paper_2502_13542_amd import harness as H
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: pytest.fail("a stream was used"))
    with pytest.raises(RuntimeError, match="cannot be captured"):
        object.__new__(H.HostCachePrefill).run_overlapped(*[None] * 7)


@pytest.mark.parametrize("fails", [False, True])
def test_streams_of_a_pass_are_joined_after_an_error_too(monkeypatch, fails):
    """Whatever ends the body, the caller's stream and the pass's own wait for every stream that it has used."""
    import contextlib
    import torch
    from paper_2502_13542_amd import harness as H
    log = []

    class Stream:
        def __init__(self, name):
            self.name = name

        def wait_stream(self, other):
            log.append(self.name + " waits for " + other.name)

    def body(self, *args):
        log.append("body")
        if fails:
            raise B.ActQKVError(-1, "refused in mid-pass")

    h = object.__new__(H.HostCachePrefill)
    outer, h.lead, h.mover, h.attender, h.writer = (Stream(x) for x in ("caller", "lead", "mover", "attender", "writer"))
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: outer)
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    monkeypatch.setattr(H.HostCachePrefill, "_run_overlapped", body)
    with pytest.raises(B.ActQKVError) if fails else contextlib.nullcontext():
        h.run_overlapped(*[None] * 7)
    assert log == ["lead waits for caller", "body", "lead waits for mover", "lead waits for attender", "lead waits for writer",
                   "caller waits for lead"]


@pytest.mark.parametrize("queues,beside,want", [
    ([2, 3, 4, 4, 3, 2, 1], [], [2, 3, 4, 1]),        # as a process's first streams are dealt
    ([4, 3, 2, 1], [], [4, 3, 2, 1]),
    ([1, 2] * 8, [], [1, 2, 1, 2]),                   # fewer queues than streams: the rest share
    ([1, 4, 4, 3], [1], [4, 3]),                      # another one than a stream's that is there
])
def test_side_streams_have_a_queue_each(monkeypatch, queues, beside, want):
    import torch
    from types import SimpleNamespace
    from paper_2502_13542_amd import harness as H
    dealt = iter(queues)
    monkeypatch.setattr(torch.cuda, "Stream", lambda device: SimpleNamespace(queue=next(dealt), synchronize=lambda: None))
    monkeypatch.setattr(torch, "empty", lambda *a, **k: None)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(H.B, "copy_bytes_at", lambda *a: None)
    monkeypatch.setattr(H, "runs_beside", lambda st, busy, src, host: st.queue != busy.queue, raising=False)
    there = [SimpleNamespace(queue=x) for x in beside]
    assert [st.queue for st in H.side_streams(len(want), "cuda", there)] == want
