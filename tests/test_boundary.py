"""Host-side tests of the C ABI (no GPU): the library loads, exports every symbol
of include/qbx.h, sizes workspaces, and rejects bad arguments before anything
reaches the device."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from paper_1207_4461_amd import _lib, inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "qbx.h")


def header_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"\b(qbx_[a-z0-9_]+)\s*\(", text)
    return sorted(set(names))


@pytest.fixture(scope="module")
def lib():
    return _lib.load()


def test_library_exports_every_declared_symbol(lib):
    names = header_functions()
    assert "qbx_layer_potential" in names and "qbx_layer_potential_adjoint" in names
    out = subprocess.run(["nm", "-D", "--defined-only", _lib.LIB_PATH], capture_output=True,
                         text=True, check=True).stdout
    exported = set(re.findall(r"\bT (qbx_[a-z0-9_]+)", out))
    missing = [n for n in names if n not in exported]
    assert not missing, missing
    for n in names:
        assert hasattr(lib, n)


def test_workspace_sizes(lib):
    n1 = lib.qbx_workspace_bytes(32, 16, 8, 4, I.EXTERIOR, 1)
    n2 = lib.qbx_workspace_bytes(64, 16, 8, 4, I.EXTERIOR, 1)
    n3 = lib.qbx_workspace_bytes(32, 16, 8, 4, I.BOTH, 3)
    assert 0 < n1 < n2 and n1 < n3 and n1 % 256 == 0
    # invalid parameters give 0
    assert lib.qbx_workspace_bytes(2, 16, 8, 4, 1, 1) == 0
    assert lib.qbx_workspace_bytes(32, 8, 8, 4, 1, 1) == 0
    assert lib.qbx_workspace_bytes(32, 16, 25, 4, 1, 1) == 0
    assert lib.qbx_workspace_bytes(32, 16, 8, 0, 1, 1) == 0
    assert lib.qbx_workspace_bytes(32, 16, 8, 4, 2, 1) == 0
    assert lib.qbx_workspace_bytes(32, 16, 8, 4, 1, 4) == 0
    assert lib.qbx_tape_bytes(32, 16, 8, I.BOTH, 3) > 0


BAD = C.c_void_p(16)  # never dereferenced: validation fails first


def _call(lib, P=8, q=16, nodes=BAD, dens=BAD, k=3.0, p=6, r=0.5, os_=4, side=1, kind=1,
          out=BAD, ws=BAD, nbytes=1 << 40):
    g = _lib.Geometry(P, q, nodes)
    return lib.qbx_layer_potential(C.byref(g), dens, k, p, r, os_, side, kind, out, None, ws,
                                   nbytes, None)


@pytest.mark.parametrize("kw", [
    dict(P=2), dict(q=8), dict(p=-1), dict(p=25), dict(k=0.0), dict(k=-1.0), dict(k=float("nan")),
    dict(k=float("inf")), dict(r=0.0), dict(r=float("nan")), dict(os_=0), dict(os_=9),
    dict(side=2), dict(kind=0), dict(kind=4), dict(nodes=None), dict(dens=None), dict(out=None),
    dict(ws=None),
])
def test_invalid_arguments_are_rejected_on_the_host(lib, kw):
    assert _call(lib, **kw) == _lib.QBX_EINVAL
    assert len(lib.qbx_last_error()) > 0


def test_small_workspace_is_rejected(lib):
    need = lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 1)
    assert _call(lib, nbytes=need - 1) == _lib.QBX_EWORKSPACE
    assert b"needed" in lib.qbx_last_error()


def test_null_geometry_and_adjoint_args(lib):
    assert lib.qbx_layer_potential(None, BAD, 1.0, 4, 0.5, 4, 1, 1, BAD, None, BAD, 1 << 40,
                                   None) == _lib.QBX_EINVAL
    g = _lib.Geometry(8, 16, BAD)
    assert lib.qbx_layer_potential_adjoint(C.byref(g), BAD, 1.0, 30, 0.5, 4, 1, 1, BAD, None,
                                           BAD, BAD, BAD, 1 << 40, None) == _lib.QBX_EINVAL
    assert lib.qbx_layer_potential_adjoint(C.byref(g), BAD, 1.0, 4, 0.5, 4, 1, 1, None, None,
                                           BAD, BAD, BAD, 1 << 40, None) == _lib.QBX_EINVAL
    assert lib.qbx_check_geometry(None, 4, 0.5, 4, 1, None, None, BAD, 1 << 40,
                                  None) == _lib.QBX_EINVAL


def test_gradient_entry_point_validates(lib):
    g = _lib.Geometry(8, 16, BAD)
    call = lambda **kw: lib.qbx_layer_potential_gradient(
        C.byref(g), kw.get("dens", BAD), kw.get("k", 3.0), kw.get("p", 6), 0.5, 4, 1, 1,
        kw.get("grad", BAD), kw.get("dn", BAD), kw.get("ws", BAD), kw.get("nbytes", 1 << 40), None)
    assert call(grad=None, dn=None) == _lib.QBX_EINVAL       # nothing to compute
    assert call(dens=None) == _lib.QBX_EINVAL
    assert call(ws=None) == _lib.QBX_EINVAL
    assert call(p=25) == _lib.QBX_EINVAL and call(k=-1.0) == _lib.QBX_EINVAL
    need = lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 1)
    assert call(nbytes=need - 1, dn=None) == _lib.QBX_EWORKSPACE
    assert lib.qbx_layer_potential_gradient(None, BAD, 1.0, 4, 0.5, 4, 1, 1, BAD, BAD, BAD,
                                            1 << 40, None) == _lib.QBX_EINVAL


def test_split_entry_point_validates(lib):
    g = _lib.Geometry(8, 16, BAD)
    call = lambda **kw: lib.qbx_layer_potential_split(
        C.byref(g), kw.get("dens", BAD), kw.get("k", 3.0), kw.get("p", 6), 0.5, 4, 1, 1,
        kw.get("gamma", 6.0), kw.get("out", BAD), kw.get("ws", BAD), kw.get("nbytes", 1 << 40),
        None)
    for bad in (dict(gamma=0.0), dict(gamma=-1.0), dict(gamma=float("nan")), dict(dens=None),
                dict(out=None), dict(ws=None), dict(p=25), dict(k=0.0)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    need = lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 1)
    assert call(nbytes=need - 1) == _lib.QBX_EWORKSPACE
    assert lib.qbx_layer_potential_split(None, BAD, 1.0, 4, 0.5, 4, 1, 1, 6.0, BAD, BAD, 1 << 40,
                                         None) == _lib.QBX_EINVAL


def test_solve_entry_point_validates(lib):
    assert lib.qbx_solve_workspace_bytes(8, 16, 6, 4, 0, 50) == 0           # both sides
    assert lib.qbx_solve_workspace_bytes(8, 16, 6, 4, 1, 0) == 0            # restart
    assert lib.qbx_solve_workspace_bytes(8, 16, 6, 4, 1, 1001) == 0
    n = lib.qbx_solve_workspace_bytes(8, 16, 6, 4, 1, 50)
    assert n > lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 3)
    assert lib.qbx_solve_workspace_bytes(8, 16, 6, 4, 1, 100) > n
    g = _lib.Geometry(8, 16, BAD)
    it, res = C.c_int(), C.c_double()

    def call(**kw):
        return lib.qbx_solve_dirichlet(
            C.byref(g), kw.get("f", BAD), 3.0, 6, 0.5, 4, kw.get("side", 1), 0.0, 1.0,
            kw.get("gamma", 0.0), kw.get("tol", 1e-14), kw.get("restart", 50),
            kw.get("max_iter", 100), kw.get("sigma", BAD), C.byref(it), C.byref(res),
            kw.get("ws", BAD), kw.get("nbytes", 1 << 40), None)

    for bad in (dict(side=0), dict(f=None), dict(sigma=None), dict(ws=None), dict(tol=0.0),
                dict(tol=float("nan")), dict(restart=0), dict(restart=1001), dict(max_iter=0),
                dict(gamma=-1.0)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    assert call(nbytes=n - 1) == _lib.QBX_EWORKSPACE
    # the adjoint system takes the same arguments and checks
    adj = lambda side=1, nbytes=1 << 40: lib.qbx_solve_dirichlet_adjoint(
        C.byref(g), BAD, 3.0, 6, 0.5, 4, side, 0.0, 1.0, 0.0, 1e-14, 50, 100, BAD, C.byref(it),
        C.byref(res), BAD, nbytes, None)
    assert adj(side=0) == _lib.QBX_EINVAL and adj(nbytes=n - 1) == _lib.QBX_EWORKSPACE


def test_solve_without_the_stored_weights(lib):
    """From 64 panels on the least workspace leaves out 24 blocks of 16 x 16 weights a panel (and an
    item of some hundred bytes); the solves refuse less, the adjoint and the split too."""
    size = (16, 6, 4, 1, 50)
    assert lib.qbx_solve_workspace_bytes_least(8, *size) == lib.qbx_solve_workspace_bytes(8, *size)
    least, full = (f(64, *size) for f in (lib.qbx_solve_workspace_bytes_least,
                                          lib.qbx_solve_workspace_bytes))
    assert 0 < full - least - 64 * 24 * 256 * 16 <= 2048
    assert lib.qbx_solve_workspace_bytes_least(64, 16, 6, 4, 0, 50) == 0
    g = _lib.Geometry(64, 16, BAD)
    for fn in (lib.qbx_solve_dirichlet, lib.qbx_solve_dirichlet_adjoint):
        for gamma in (0.0, 6.0):
            assert fn(C.byref(g), BAD, 3.0, 6, 0.5, 4, 1, 0.0, 1.0, gamma, 1e-14, 50, 100, BAD,
                      None, None, BAD, least - 1, None) == _lib.QBX_EWORKSPACE


def test_ext_entry_point_validates(lib):
    g = _lib.Geometry(8, 16, BAD)

    def call(dipole=0, rule=0, dens=BAD, out=BAD, ws=BAD, nbytes=1 << 40, use_opt=True):
        opt = _lib.ForwardOptions(dipole, rule)
        return lib.qbx_layer_potential_ext(C.byref(g), dens, 3.0, 6, 0.5, 4, 1, 2,
                                           C.byref(opt) if use_opt else None, out, ws, nbytes,
                                           None)

    for bad in (dict(dipole=2), dict(dipole=-1), dict(rule=2), dict(dens=None), dict(out=None),
                dict(ws=None)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    need = lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 2)
    assert call(nbytes=need - 1) == _lib.QBX_EWORKSPACE
    assert call(nbytes=need - 1, use_opt=False) == _lib.QBX_EWORKSPACE


def test_split_adjoint_entry_point_validates(lib):
    g = _lib.Geometry(8, 16, BAD)

    def call(**kw):
        return lib.qbx_layer_potential_split_adjoint(
            C.byref(g), kw.get("dens", BAD), 3.0, 6, 0.5, 4, 1, 1, kw.get("gamma", 6.0),
            kw.get("cot", BAD), kw.get("gd", BAD), kw.get("gn", None), kw.get("ws", BAD),
            kw.get("nbytes", 1 << 40), None)

    for bad in (dict(gamma=0.0), dict(dens=None), dict(cot=None), dict(gd=None), dict(ws=None),
                dict(gd=None, gn=None), dict(gn=BAD, ws=None)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    assert call(nbytes=lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 1) - 1) == _lib.QBX_EWORKSPACE


def test_timer_class_count_matches_header():
    """qbx_kernel_timer_read writes QBX_TIMER_CLASSES entries into caller arrays: the
    binding's constant must be the header's."""
    hdr = open(os.path.join(os.path.dirname(__file__), "..", "include", "qbx.h")).read()
    assert int(re.search(r"#define QBX_TIMER_CLASSES (\d+)", hdr).group(1)) == _lib.QBX_TIMER_CLASSES


def test_strerror(lib):
    for code in (0, -1, -2, -3, -4, -5, -6):
        assert len(lib.qbx_strerror(code)) > 3
    assert lib.qbx_strerror(-99) == b"unknown error"


def test_signed_area_host_and_orientation(lib):
    pb = I.small(n_panels=12)
    nodes = np.ascontiguousarray(pb.nodes)
    area = C.c_double()
    assert lib.qbx_signed_area_host(nodes.ctypes.data, 12, C.byref(area)) == _lib.QBX_OK
    # area enclosed by r(t) = 1 + 0.15 cos(3t + 0.3): pi (1 + 0.15^2 / 2)
    assert abs(area.value - np.pi * (1 + 0.15**2 / 2)) < 1e-12
    rev = np.ascontiguousarray(nodes[::-1, ::-1, :])     # same curve, clockwise
    assert lib.qbx_signed_area_host(rev.ctypes.data, 12, C.byref(area)) == _lib.QBX_EORIENT
    assert area.value < 0
    assert lib.qbx_signed_area_host(None, 12, None) == _lib.QBX_EINVAL
    assert lib.qbx_signed_area_host(nodes.ctypes.data, 2, None) == _lib.QBX_EINVAL


def test_debug_hooks_validate(lib):
    assert lib.qbx_debug_hankel01(None, 4, None, None, None) == _lib.QBX_EINVAL
    assert lib.qbx_debug_besselj(BAD, 4, 99, BAD, None) == _lib.QBX_EINVAL


def test_principal_value_validation(lib):
    assert lib.qbx_principal_value(None, None, 8, 0, 1, BAD, None) == _lib.QBX_EINVAL
    assert lib.qbx_principal_value(BAD, None, 2, 0, 1, BAD, None) == _lib.QBX_EINVAL
    assert lib.qbx_principal_value(BAD, None, 8, 3, 1, BAD, None) == _lib.QBX_EINVAL
    assert lib.qbx_principal_value(BAD, None, 8, 1, 2, BAD, None) == _lib.QBX_EINVAL


def _items(n=3):
    its = (_lib.BatchItem * n)()
    for i in range(n):
        it = its[i]
        it.node_offset, it.density_offset, it.out_offset = 8 * i, 128 * i, 256 * i
        it.n_panels, it.p, it.kind, it.side, it.k, it.r = 8, 6, 1, 0, 3.0, 0.5
    return its


def test_batched_validation(lib):
    its = _items()
    n = lib.qbx_batched_workspace_bytes(its, 3, 4)
    assert n > 0 and n % 256 == 0
    assert lib.qbx_batched_tape_bytes(its, 3) > 0
    assert lib.qbx_batched_workspace_bytes(its, 0, 4) == 0
    assert lib.qbx_batched_workspace_bytes(its, 3, 0) == 0
    for field, bad in (("n_panels", 2), ("p", 25), ("kind", 0), ("side", 5), ("k", -1.0),
                       ("r", 0.0), ("node_offset", -1)):
        its = _items()
        setattr(its[1], field, bad)
        assert lib.qbx_batched_workspace_bytes(its, 3, 4) == 0
        assert lib.qbx_layer_potential_batched(its, 3, BAD, BAD, BAD, None, 4, BAD, 1 << 40,
                                               None) == _lib.QBX_EINVAL
    its = _items()
    assert lib.qbx_layer_potential_batched(its, 3, None, BAD, BAD, None, 4, BAD, 1 << 40,
                                           None) == _lib.QBX_EINVAL
    assert lib.qbx_layer_potential_batched(its, 3, BAD, BAD, BAD, None, 4, BAD, 10,
                                           None) == _lib.QBX_EWORKSPACE
    assert lib.qbx_layer_potential_batched_adjoint(its, 3, BAD, BAD, None, None, BAD, BAD, 4, BAD,
                                                   1 << 40, None) == _lib.QBX_EINVAL


def test_tuning_roundtrip_and_validation(lib):
    t0 = _lib.Tuning()
    assert lib.qbx_get_tuning(C.byref(t0)) == _lib.QBX_OK
    assert t0.forward_waves >= 256 and 0.125 <= t0.batch_grid_scale <= 8
    fields = [f for f, _ in _lib.Tuning._fields_]
    t = _lib.Tuning(*[getattr(t0, f) for f in fields])
    assert t0.fused_tiles >= 256 and 1 <= t0.batch_fused_chunks <= 64
    try:
        n_before = lib.qbx_workspace_bytes(256, 16, 8, 4, 1, 1)
        t.forward_waves = 1 << 20          # more source splits -> larger partial buffers
        assert lib.qbx_set_tuning(C.byref(t)) == _lib.QBX_OK
        t1 = _lib.Tuning()
        lib.qbx_get_tuning(C.byref(t1))
        assert t1.forward_waves == 1 << 20
        assert lib.qbx_workspace_bytes(256, 16, 8, 4, 1, 1) > n_before
        t.fused_tiles = 1 << 14
        t.batch_fused_chunks = 7
        assert lib.qbx_set_tuning(C.byref(t)) == _lib.QBX_OK
        lib.qbx_get_tuning(C.byref(t1))
        assert (t1.fused_tiles, t1.batch_fused_chunks) == (1 << 14, 7)
        # the fused adjoint's partial-sum bound: default 2^31; a smaller bound means
        # taller tiles and so a smaller workspace (star1024 sizes: 1024 panels, S)
        assert t0.fused_part_bytes == 2.0 ** 31
        n_wide = lib.qbx_workspace_bytes(1024, 16, 16, 4, 1, 1)
        t.fused_part_bytes = 1 << 20
        assert lib.qbx_set_tuning(C.byref(t)) == _lib.QBX_OK
        lib.qbx_get_tuning(C.byref(t1))
        assert t1.fused_part_bytes == 1 << 20
        assert lib.qbx_workspace_bytes(1024, 16, 16, 4, 1, 1) < n_wide
        for field, bad in (("forward_waves", 255), ("tape_waves", 1 << 23), ("adjoint_waves", 0),
                           ("batch_adjoint_tasks", -5), ("batch_grid_scale", 0.1),
                           ("batch_grid_scale", 9.0), ("batch_grid_scale", float("nan")),
                           ("fused_tiles", 100), ("fused_tiles", 1 << 23),
                           ("batch_fused_chunks", 0), ("batch_fused_chunks", 65),
                           ("fused_part_bytes", 4095.0), ("fused_part_bytes", 2.0 ** 41),
                           ("fused_part_bytes", float("nan"))):
            tb = _lib.Tuning(*[getattr(t0, f) for f in fields])
            setattr(tb, field, bad)
            assert lib.qbx_set_tuning(C.byref(tb)) == _lib.QBX_EINVAL
        assert lib.qbx_set_tuning(None) == _lib.QBX_EINVAL
        assert lib.qbx_get_tuning(None) == _lib.QBX_EINVAL
    finally:
        assert lib.qbx_set_tuning(C.byref(t0)) == _lib.QBX_OK


def _autotune(lib, g, dens=BAD, p=4, passes=2, fields=None, cache=None, ws=BAD, nbytes=1 << 40):
    fields = _lib.QBX_TUNE_ALL if fields is None else fields
    return lib.qbx_autotune(C.byref(g), dens, 1.0, p, 0.5, 4, 1, 1, passes, fields, cache, None,
                            ws, nbytes, None)


def test_autotune_validation(lib):
    g = _lib.Geometry(8, 16, BAD)
    ALL = _lib.QBX_TUNE_ALL
    assert _autotune(lib, g, p=30) == _lib.QBX_EINVAL
    assert _autotune(lib, g, dens=None) == _lib.QBX_EINVAL
    assert _autotune(lib, g, passes=0) == _lib.QBX_EINVAL
    for bad in (0, 16, -1):   # fields: a nonzero combination of the four bits
        assert _autotune(lib, g, fields=bad) == _lib.QBX_EINVAL
    assert _autotune(lib, g, ws=None) == _lib.QBX_EINVAL
    need = lib.qbx_autotune_workspace_bytes(8, 16, 4, 4, 1, 1)
    assert need >= lib.qbx_workspace_bytes(8, 16, 4, 4, 1, 1) and need % 256 == 0
    assert lib.qbx_autotune_workspace_bytes(2, 16, 4, 4, 1, 1) == 0
    assert _autotune(lib, g, nbytes=need - 1) == _lib.QBX_EWORKSPACE
    its = _items()
    nb = lib.qbx_autotune_batched_workspace_bytes(its, 3, 4)
    assert nb >= lib.qbx_batched_workspace_bytes(its, 3, 4) and nb % 256 == 0

    def batched(n=3, passes=2, fields=ALL, ws=BAD, nbytes=1 << 40):
        return lib.qbx_autotune_batched(its, n, BAD, BAD, 4, passes, fields, None, None, ws,
                                        nbytes, None)

    assert batched(passes=0) == _lib.QBX_EINVAL
    assert batched(n=0) == _lib.QBX_EINVAL
    assert batched(fields=0) == _lib.QBX_EINVAL
    assert batched(ws=None) == _lib.QBX_EINVAL
    assert batched(nbytes=nb - 1) == _lib.QBX_EWORKSPACE
    its[0].p = 99
    assert batched() == _lib.QBX_EINVAL
    assert lib.qbx_autotune_batched_workspace_bytes(its, 3, 4) == 0


def test_autotune_leaves_shapes_that_do_not_act(lib):
    """With panel expansions (512 panels, r = 1/2) the passes without a tape run no kernel that
    forward_waves or fused_tiles shapes: nothing is timed (no device is needed) and the fields
    keep their values, which are none of the candidates."""
    fields = [n for n, _ in _lib.Tuning._fields_]
    t0, best = _lib.Tuning(), _lib.Tuning()
    assert lib.qbx_get_tuning(C.byref(t0)) == _lib.QBX_OK
    try:
        t = _lib.Tuning(*[getattr(t0, f) for f in fields])
        t.forward_waves, t.fused_tiles, t.batch_grid_scale, t.batch_fused_chunks = 5000, 3000, 1.5, 5
        assert lib.qbx_set_tuning(C.byref(t)) == _lib.QBX_OK
        what = _lib.QBX_TUNE_FORWARD | _lib.QBX_TUNE_FUSED
        g = _lib.Geometry(512, 16, BAD)
        assert lib.qbx_autotune(C.byref(g), BAD, 1.0, 8, 0.5, 4, 1, 1, 2, what, None, C.byref(best),
                                BAD, 1 << 40, None) == _lib.QBX_OK
        assert all(getattr(best, f) == getattr(t, f) for f in fields)
        its = (_lib.BatchItem * 2)(*[_lib.BatchItem(512 * i, 8192 * i, 8192 * i, 512, 8, 1, 1, 3.0,
                                                    0.5) for i in range(2)])
        assert lib.qbx_autotune_batched(its, 2, BAD, BAD, 4, 2, what, None, C.byref(best), BAD,
                                        1 << 40, None) == _lib.QBX_OK
        assert all(getattr(best, f) == getattr(t, f) for f in fields)
    finally:
        assert lib.qbx_set_tuning(C.byref(t0)) == _lib.QBX_OK


def test_autotune_workspace_covers_every_candidate(lib):
    """The autotuner's workspace query holds the library workspace of every
    candidate shape (the library's own size depends on the tuning)."""
    t0 = _lib.Tuning()
    assert lib.qbx_get_tuning(C.byref(t0)) == _lib.QBX_OK
    need = lib.qbx_autotune_workspace_bytes(300, 16, 12, 4, 0, 3)
    try:
        for w in (2048, 4096, 8192, 16384, 32768, 65536, 131072):
            for f in (2048, 4096, 8192, 16384, 32768):
                t = _lib.Tuning.from_buffer_copy(t0)
                t.forward_waves = t.tape_waves = t.adjoint_waves = w
                t.fused_tiles = f
                assert lib.qbx_set_tuning(C.byref(t)) == _lib.QBX_OK
                assert lib.qbx_workspace_bytes(300, 16, 12, 4, 0, 3) < need
    finally:
        assert lib.qbx_set_tuning(C.byref(t0)) == _lib.QBX_OK


def _explicit(lib, n_src=100, n_ctr=20, p=6, kind=1, k=3.0, xy=BAD, nu=BAD, q=BAD, cxy=BAD,
              cr=BAD, cd=BAD, out=BAD, ws=BAD, nbytes=1 << 40):
    return lib.qbx_apply_explicit(n_src, xy, nu, q, n_ctr, cxy, cr, cd, k, p, kind, out, None, ws,
                                  nbytes, None)


def test_explicit_sizes_and_validation(lib):
    n1 = lib.qbx_explicit_workspace_bytes(1000, 100, 8, 1)
    n2 = lib.qbx_explicit_workspace_bytes(1000, 100, 8, 3)
    assert 0 < n1 < n2 and n1 % 256 == 0
    assert lib.qbx_explicit_workspace_bytes(0, 100, 8, 1) == 0
    assert lib.qbx_explicit_workspace_bytes(10, 0, 8, 1) == 0
    assert lib.qbx_explicit_workspace_bytes(10, 10, 25, 1) == 0
    assert lib.qbx_explicit_workspace_bytes(10, 10, 8, 0) == 0
    assert lib.qbx_explicit_tape_bytes(10, 3) == 10 * 2 * 4 * 16
    assert lib.qbx_explicit_tape_bytes(0, 3) == 0
    for kw in (dict(n_src=0), dict(n_ctr=0), dict(p=-1), dict(p=25), dict(kind=4), dict(k=0.0),
               dict(k=float("nan")), dict(xy=None), dict(q=None), dict(cxy=None), dict(cr=None),
               dict(cd=None), dict(out=None), dict(ws=None), dict(kind=2, nu=None)):
        assert _explicit(lib, **kw) == _lib.QBX_EINVAL, kw
    assert _explicit(lib, kind=1, nu=None, nbytes=10) == _lib.QBX_EWORKSPACE
    assert lib.qbx_apply_explicit_adjoint(10, BAD, BAD, BAD, 5, BAD, BAD, BAD, 1.0, 4, 1, None,
                                          None, BAD, BAD, BAD, BAD, BAD, BAD, BAD, 1 << 40,
                                          None) == _lib.QBX_EINVAL


def test_differentiable_solve_requires_convergence():
    """The differentiable Dirichlet solve refuses a GMRES run that max_iter cut short."""
    from paper_1207_4461_amd import qbx
    qbx._require_converged("solve", 40, 5e-13, 1e-14)          # within 100 tol
    for bad in (2e-12, float("nan"), float("inf")):
        with pytest.raises(RuntimeError, match="GMRES stopped"):
            qbx._require_converged("solve", 1000, bad, 1e-14)


def test_noalloc_entry_point_validates(lib):
    g = _lib.Geometry(8, 16, BAD)
    call = lambda gp=C.byref(g), **kw: lib.qbx_layer_potential_noalloc(
        gp, kw.get("dens", BAD), kw.get("k", 3.0), kw.get("p", 6), 0.5, kw.get("os_", 4),
        kw.get("side", 1), kw.get("kind", 1), kw.get("out", BAD), None)
    for bad in (dict(dens=None), dict(out=None), dict(p=25), dict(k=0.0), dict(os_=0),
                dict(side=2), dict(kind=4)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    assert call(gp=None) == _lib.QBX_EINVAL
    # star4096 (4096 panels, both sides, S+D, p = 20) needs more than the static
    # scratch holds: refused on the host, before any device call
    big = _lib.Geometry(4096, 16, BAD)
    assert lib.qbx_layer_potential_noalloc(C.byref(big), BAD, 100.0, 20, 0.5, 4, 0, 3, BAD,
                                           None) == _lib.QBX_EWORKSPACE
    assert b"static scratch" in lib.qbx_last_error()
    assert _lib.QBX_STATIC_SCRATCH_BYTES == 64 << 20


def test_gradient_principal_value_validates(lib):
    g = _lib.Geometry(8, 16, BAD)
    call = lambda gp=C.byref(g), **kw: lib.qbx_gradient_principal_value(
        gp, kw.get("dens", BAD), kw.get("side", 1), kw.get("kind", 3), kw.get("grad", BAD),
        kw.get("dn", BAD), kw.get("gpv", BAD), kw.get("dpv", BAD), None)
    for bad in (dict(side=2), dict(kind=0), dict(kind=4), dict(dens=None),
                dict(grad=None), dict(dpv=None), dict(grad=None, gpv=None, dn=None, dpv=None)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    assert call(gp=None) == _lib.QBX_EINVAL
    assert call(gp=C.byref(_lib.Geometry(2, 16, BAD))) == _lib.QBX_EINVAL
    assert call(gp=C.byref(_lib.Geometry(8, 8, BAD))) == _lib.QBX_EINVAL
    assert call(gp=C.byref(_lib.Geometry(8, 16, None))) == _lib.QBX_EINVAL


def test_explicit_gradient_validates(lib):
    call = lambda **kw: lib.qbx_apply_explicit_gradient(
        kw.get("ns", 10), BAD, kw.get("nu", BAD), BAD, kw.get("nc", 4), BAD, BAD, BAD,
        kw.get("k", 2.0), kw.get("p", 5), kw.get("kind", 3), kw.get("grad", BAD), BAD,
        kw.get("nbytes", 1 << 40), None)
    for bad in (dict(ns=0), dict(nc=0), dict(p=25), dict(kind=4), dict(k=0.0), dict(grad=None),
                dict(nu=None)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    need = lib.qbx_explicit_workspace_bytes(10, 4, 5, 3)
    assert call(nbytes=need - 1) == _lib.QBX_EWORKSPACE


def test_expansion_entry_points_validate(lib):
    g = _lib.Geometry(8, 16, BAD)
    call = lambda gp=C.byref(g), **kw: lib.qbx_expansion_coefficients(
        gp, kw.get("dens", BAD), kw.get("k", 3.0), kw.get("p", 6), 0.5, 4, kw.get("side", 1),
        kw.get("kind", 3), kw.get("coef", BAD), None, None, kw.get("ws", BAD),
        kw.get("nbytes", 1 << 40), None)
    for bad in (dict(dens=None), dict(coef=None), dict(ws=None), dict(p=25), dict(k=0.0),
                dict(side=2), dict(kind=4)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    assert call(gp=None) == _lib.QBX_EINVAL
    need = lib.qbx_expansion_workspace_bytes(8, 16, 6, 4, 1, 3)
    assert need > 0 and lib.qbx_expansion_workspace_bytes(8, 16, 25, 4, 1, 3) == 0
    assert call(nbytes=need - 1) == _lib.QBX_EWORKSPACE
    ev = lambda **kw: lib.qbx_evaluate_expansions(
        kw.get("nc", 10), kw.get("cxy", BAD), BAD, kw.get("k", 2.0), kw.get("p", 4),
        kw.get("kind", 1), kw.get("nt", 5), BAD, kw.get("idx", BAD), BAD, None)
    for bad in (dict(nc=0), dict(nt=-1), dict(p=25), dict(k=-1.0), dict(kind=0), dict(cxy=None),
                dict(idx=None)):
        assert ev(**bad) == _lib.QBX_EINVAL, bad
    assert ev(nt=0, cxy=None) == _lib.QBX_OK     # nothing to do
    asg = lambda **kw: lib.qbx_assign_centers(kw.get("nc", 10), BAD, kw.get("r", BAD),
                                              kw.get("nt", 5), BAD, kw.get("slack", 1.0),
                                              BAD, None)
    for bad in (dict(nc=0), dict(nt=-1), dict(slack=0.0), dict(slack=float("nan")),
                dict(r=None)):
        assert asg(**bad) == _lib.QBX_EINVAL, bad


def test_workspace_size_follows_the_tuning(lib):
    """qbx_workspace_bytes depends on the tuning; a workspace sized under a smaller
    tuning is refused under a larger one (before anything reaches the device)."""
    t0 = _lib.Tuning()
    assert lib.qbx_get_tuning(C.byref(t0)) == _lib.QBX_OK
    try:
        sizes = []
        for w in (2048, 131072):
            t = _lib.Tuning.from_buffer_copy(t0)
            t.forward_waves = t.tape_waves = t.adjoint_waves = w
            assert lib.qbx_set_tuning(C.byref(t)) == _lib.QBX_OK
            sizes.append(lib.qbx_workspace_bytes(64, 16, 10, 4, 0, 3))
        assert sizes[0] < sizes[1]
        g = _lib.Geometry(64, 16, BAD)
        rc = lib.qbx_layer_potential(C.byref(g), BAD, 3.0, 10, 0.5, 4, 0, 3, BAD, None, BAD,
                                     sizes[0], None)
        assert rc == _lib.QBX_EWORKSPACE
    finally:
        assert lib.qbx_set_tuning(C.byref(t0)) == _lib.QBX_OK


def test_autotune_cache_file_errors(lib, tmp_path):
    """A malformed or unreadable cache file, and a device query without a device, give
    their codes; every case returns before any device memory is touched."""
    g = _lib.Geometry(8, 16, BAD)
    bad_dir = str(tmp_path).encode()   # a directory: not a cache file
    rc = _autotune(lib, g, cache=bad_dir, ws=None)
    # without a GPU the cache key's device query fails first
    assert rc in (_lib.QBX_EIO, _lib.QBX_EDEVICE)
    if rc == _lib.QBX_EDEVICE:
        assert b"device" in lib.qbx_last_error()


def test_device_errors_are_reported_without_a_gpu(lib):
    """QBX_EDEVICE from entry points whose arguments pass validation, forced on a
    machine with no GPU (the first launch fails); the message names the step."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present: device errors cannot be forced from the host")
    g = _lib.Geometry(8, 16, BAD)
    n = lib.qbx_workspace_bytes(8, 16, 6, 4, 1, 1)
    calls = {
        "forward": lambda: lib.qbx_layer_potential(C.byref(g), BAD, 3.0, 6, 0.5, 4, 1, 1, BAD,
                                                   None, BAD, n, None),
        "split": lambda: lib.qbx_layer_potential_split(C.byref(g), BAD, 3.0, 6, 0.5, 4, 1, 1, 6.0,
                                                       BAD, BAD, n, None),
        "adjoint": lambda: lib.qbx_layer_potential_adjoint(C.byref(g), BAD, 3.0, 6, 0.5, 4, 1, 1,
                                                           BAD, None, BAD, BAD, BAD, n, None),
        "autotune cache key": lambda: _autotune(lib, g, cache=b"/nonexistent/qbx_cache.txt"),
    }
    for name, call in calls.items():
        rc = call()
        assert rc == _lib.QBX_EDEVICE, (name, rc, lib.qbx_last_error())
        assert len(lib.qbx_last_error()) > 10, name
    assert lib.qbx_strerror(_lib.QBX_EIO) == b"autotuner cache file error"


def test_solve_node_gradient_validation(lib):
    g = _lib.Geometry(8, 16, BAD)
    need = lib.qbx_solve_node_gradient_workspace_bytes(8, 16, 6, 4)
    assert need >= lib.qbx_workspace_bytes(8, 16, 6, 4, 0, 3) and need % 256 == 0
    assert lib.qbx_solve_node_gradient_workspace_bytes(8, 16, 99, 4) == 0

    def call(side=1, sig=BAD, lam=BAD, gn=BAD, gamma=0.0, alpha=(0.0, 1.0), ws=BAD,
             nbytes=need):
        return lib.qbx_solve_dirichlet_node_gradient(C.byref(g), sig, lam, 3.0, 6, 0.5, 4, side,
                                                     alpha[0], alpha[1], gamma, gn, ws, nbytes,
                                                     None)

    for bad in (dict(side=0), dict(sig=None), dict(lam=None), dict(gn=None), dict(gamma=-1.0),
                dict(gamma=float("nan")), dict(alpha=(float("inf"), 0.0)), dict(ws=None)):
        assert call(**bad) == _lib.QBX_EINVAL, bad
    assert call(nbytes=need - 1) == _lib.QBX_EWORKSPACE
