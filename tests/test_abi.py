"""The C-ABI library loads and exports every symbol the header declares (no GPU needed)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2505_13254_amd", "libheterospec.so")


def _declared():
    text = open(os.path.join(ROOT, "include", "heterospec.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(hs_[a-z_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        import sys
        sys.path.insert(0, ROOT)
        from paper_2505_13254_amd.build import build
        build(verbose=False)
    return ctypes.CDLL(LIB)


def test_header_declares_the_four_calls():
    names = _declared()
    for n in ("hs_draft_entropy_topk", "hs_tree_prune", "hs_tree_attention", "hs_verify_accept"):
        assert n in names and n + "_workspace" in names


def test_every_declared_symbol_is_exported(lib):
    for n in _declared():
        assert hasattr(lib, n), n


def test_binding_signatures_cover_the_header():
    from paper_2505_13254_amd import binding
    assert binding.exported_symbols() == _declared()


def test_host_side_calls(lib):
    lib.hs_version.restype = ctypes.c_char_p
    lib.hs_status_string.restype = ctypes.c_char_p
    lib.hs_last_error.restype = ctypes.c_char_p
    assert lib.hs_version().decode()[0].isdigit()
    assert b"workspace" in lib.hs_status_string(4)
    # workspace queries are plain host arithmetic
    f = lib.hs_draft_entropy_topk_workspace
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int32] * 3
    assert f(61, 128256, 10) > 0 and f(61, 128256, 10) % 256 == 0 and f(0, 128256, 10) == 0
    g = lib.hs_tree_attention_workspace
    g.restype = ctypes.c_size_t
    g.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                  ctypes.c_int]
    assert g(1, 61, 2048, 32, 8, 128, 1) % 256 == 0


def test_argument_validation_needs_no_gpu(lib):
    # errors are found on the host before anything is launched
    fn = lib.hs_draft_entropy_topk
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_float] + \
                  [ctypes.c_void_p] * 6 + [ctypes.c_size_t, ctypes.c_void_p]
    lib.hs_last_error.restype = ctypes.c_char_p
    assert fn(None, 100, 4, 100, 0, 1.0, None, None, None, None, None, None, 0, None) == 2       # K = 0
    assert b"K=0" in lib.hs_last_error()
    assert fn(None, 100, 4, 100, 65, 1.0, None, None, None, None, None, None, 0, None) == 3      # K > 64
    assert fn(None, 10, 4, 100, 5, 1.0, None, None, None, None, None, None, 0, None) == 2        # stride < V
    assert fn(None, 100, 4, 100, 5, 1.0, None, None, None, None, None, None, 0, None) == 1       # NULL logits
    assert fn(None, 100, 0, 100, 5, 1.0, None, None, None, None, None, None, 0, None) == 0       # R = 0: no-op
    pr = lib.hs_tree_prune
    pr.restype = ctypes.c_int
    pr.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 2 + [ctypes.c_void_p] * 10 + [ctypes.c_size_t, ctypes.c_void_p]
    assert pr(None, None, None, -1, 0, *([None] * 10), 0, None) == 2
    assert pr(None, None, None, 2, 5, *([None] * 10), 0, None) == 1
    at = lib.hs_tree_attention
    at.restype = ctypes.c_int
    at.argtypes = [ctypes.c_void_p] * 10 + [ctypes.c_int32] * 4 + [ctypes.c_int, ctypes.c_float] + \
                  [ctypes.c_void_p] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    assert at(*([None] * 10), 1, 6, 4, 128, 1, 0.1, None, None, None, 0, None) == 2             # Hq % Hkv
    assert at(*([None] * 10), 1, 8, 4, 96, 1, 0.1, None, None, None, 0, None) == 3              # D = 96
    hno = (ctypes.c_int32 * 2)(0, 2000)
    hpo = (ctypes.c_int64 * 2)(0, 10)
    dummy = ctypes.c_void_p(256)
    assert at(dummy, dummy, dummy, dummy, dummy, dummy, dummy, dummy, ctypes.cast(hno, ctypes.c_void_p),
              ctypes.cast(hpo, ctypes.c_void_p), 1, 8, 4, 128, 1, 0.1, dummy, None, None, 0, None) == 3  # > 1024 rows
    va = lib.hs_verify_accept
    va.restype = ctypes.c_int
    va.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int64] + [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 3 + \
                  [ctypes.c_int, ctypes.c_float, ctypes.c_void_p, ctypes.c_int32] + [ctypes.c_void_p] * 4 + \
                  [ctypes.c_size_t, ctypes.c_void_p]
    assert va(None, None, 10, None, None, None, 1, 4, 10, 0, 1.0, None, 0, None, None, None, None, 0, None) == 2  # max_depth
    assert va(None, None, 10, None, None, None, 1, 4, 10, 7, 1.0, None, 3, None, None, None, None, 0, None) == 2  # mode


def test_accept_workspace_depends_on_the_mode(lib):
    q = lib.hs_verify_accept_workspace
    q.restype, q.argtypes = ctypes.c_size_t, [ctypes.c_int32] * 3
    qm = lib.hs_verify_accept_workspace_mode
    qm.restype, qm.argtypes = ctypes.c_size_t, [ctypes.c_int32] * 3 + [ctypes.c_int]
    greedy, ratio, point = (qm(1, 61, 128256, m) for m in (0, 1, 2))
    assert greedy == point < ratio == q(1, 61, 128256)
    assert ratio - greedy >= 61 * 128256 * 8                  # a pair of floats per row and token
    assert greedy < 64 * 1024 * 1024 and greedy % 256 == 0 and ratio % 256 == 0
    assert qm(1, 5000, 128256, 1) - qm(1, 5000, 128256, 0) < 1 << 20   # too many rows for the sorted residual
    # a workspace of the greedy size is refused by the ratio rule and the other way round it is fine;
    # both are decided on the host
    va = lib.hs_verify_accept
    va.restype = ctypes.c_int
    va.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int64] + [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 3 + \
                  [ctypes.c_int, ctypes.c_float, ctypes.c_void_p, ctypes.c_int32] + [ctypes.c_void_p] * 4 + \
                  [ctypes.c_size_t, ctypes.c_void_p]
    d = ctypes.c_void_p(256)
    assert va(d, d, 128256, d, d, d, 1, 61, 128256, 1, 1.0, d, 6, d, d, d, d, greedy, None) == 4
    assert va(d, d, 128256, d, d, d, 1, 61, 128256, 0, 1.0, d, 6, d, d, d, d, greedy - 256, None) == 4


@pytest.mark.parametrize("V", [1024, 8000, 32000, 50257, 128256, 262144])
def test_a_workspace_for_many_rows_holds_fewer(lib, V):
    """Callers size a workspace for their largest step: the queries never fall as rows are added."""
    f = lib.hs_draft_entropy_topk_workspace
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int32] * 3
    qm = lib.hs_verify_accept_workspace_mode
    qm.restype, qm.argtypes = ctypes.c_size_t, [ctypes.c_int32] * 3 + [ctypes.c_int]
    for need in [lambda r: f(r, V, 10), lambda r: qm(1, r, V, 0), lambda r: qm(1, r, V, 1)]:
        sizes = [need(r) for r in range(1, 700)]
        assert sizes == sorted(sizes)


@pytest.mark.parametrize("B,NN,V,depth", [(1, 65536, 8, 1), (1, 65536, 32000, 1), (1000, 65536, 128256, 4), (70000, 70000, 100, 2),
                                          (1, 1 << 30, 600, 1)])
def test_accept_calls_of_too_many_rows_are_refused_whatever_their_shape(lib, B, NN, V, depth):
    """More than 65535 rows to scan (the ratio rule scans twice the rows): HS_ERR_UNSUPPORTED on the host, for shapes that the
    greedy walk would take row by row along the paths as well."""
    va = lib.hs_verify_accept
    va.restype = ctypes.c_int
    va.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int64] + [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 3 + \
                  [ctypes.c_int, ctypes.c_float, ctypes.c_void_p, ctypes.c_int32] + [ctypes.c_void_p] * 4 + \
                  [ctypes.c_size_t, ctypes.c_void_p]
    d = ctypes.c_void_p(256)
    for mode, rows in [(0, NN), (1, 32768), (1, NN), (2, NN)]:
        assert va(d, d, V, d, d, d, B, rows, V, mode, 1.0, d, depth, d, d, d, d, 1 << 62, None) == 3, mode


@pytest.mark.parametrize("missing", ["torch", "compiler", "headers"])
def test_the_library_is_linked_where_the_native_module_cannot_be(tmp_path, monkeypatch, missing):
    """libheterospec.so needs hipcc and nothing else: what the binding's module needs may be absent (the compile and link
    lines are stood in for, the order and what is raised are the build's own)."""
    from paper_2505_13254_amd import build as B
    tool = tmp_path / "hipcc"
    tool.write_text('#!/bin/sh\nwhile [ "$1" != "-o" ]; do shift; done\necho built > "$2"\n')
    tool.chmod(0o755)
    for name, value in [("PKG", str(tmp_path)), ("LIB", str(tmp_path / "lib.so")), ("MARSHAL", str(tmp_path / "_m.so")), ("hipcc", lambda: str(tool))]:
        monkeypatch.setattr(B, name, value)
    def no_torch():
        raise ImportError("No module named 'torch'")
    monkeypatch.setattr(B, "marshal_command", {"torch": no_torch, "compiler": lambda: [str(tmp_path / "no-such-compiler")],
                                               "headers": lambda: ["/bin/sh", "-c", "echo Python.h: No such file; exit 1"]}[missing])
    with pytest.raises(RuntimeError, match="marshal|native module"):
        B.build(verbose=False)
    assert (tmp_path / "lib.so").read_text() == "built\n" and not (tmp_path / "_m.so").exists()
    (tmp_path / "lib.so").unlink()
    B.build_library(verbose=False)
    assert (tmp_path / "lib.so").exists()


def test_adaptive_policy_on_the_host_matches_the_worked_table(lib):
    """hs_adaptive_policy (host arithmetic only) against the hand-worked Section 4.3 table of the figure example."""
    f = lib.hs_adaptive_policy
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int32, ctypes.c_void_p] + [ctypes.c_int32] * 4 + [ctypes.c_void_p, ctypes.c_void_p]
    gamma = (ctypes.c_float * 3)(0.3, 0.6, 1.0)
    rows = [tuple(int(x) for x in line.split()) for line in
            open(os.path.join(ROOT, "tests", "golden", "control_figure_example.txt")) if line[0] != "#"]
    assert len(rows) == 8
    for b, _delta, dp, npr in rows:
        got_d, got_n = ctypes.c_int32(-1), ctypes.c_int32(-1)
        assert f(b, ctypes.cast(gamma, ctypes.c_void_p), 3, 3, 5, 20, ctypes.byref(got_d), ctypes.byref(got_n)) == 0
        assert (got_d.value, got_n.value) == (dp, npr), b
    assert f(-1, ctypes.cast(gamma, ctypes.c_void_p), 3, 3, 5, 20, ctypes.byref(got_d), ctypes.byref(got_n)) == 2
    assert f(0, None, 3, 3, 5, 20, ctypes.byref(got_d), ctypes.byref(got_n)) == 1
