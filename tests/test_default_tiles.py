"""The default tile on the host: a box is refused only if no tile fits it.

pic_create checks a configuration before its first HIP call, so a box whose
tile does not suit it or does not fit the LDS fails with PIC_E_INVALID also
where there is no GPU (a box that is taken fails there with PIC_E_HIP).
Windows, r-z walls, TRISTAN, the int64 current, partly asked tiles and long
intervals: each leaves the default less room than a plain periodic box."""
import ctypes
import math
import os
import random

import pytest


def _taken(pic, **kw):
    cfg = pic.Config(**kw).c()
    h = ctypes.c_void_p()
    L = pic.lib()
    rc = L.pic_create(ctypes.byref(cfg), None, ctypes.byref(h))
    if rc == 0:
        L.pic_destroy(h)
    return rc != pic.PIC_E_INVALID


@pytest.fixture(scope="module")
def pic():
    from paper_1503_00276_amd import pic

    if not os.path.exists(pic.LIB_PATH):
        pytest.skip("libpic.so not built (run __graft_entry__.build())")
    return pic


def _box(nx, courant=0.95, **kw):
    return dict(ndim=len(nx), nx=nx, dx=(0.2,) * len(nx), dt=courant * 0.2 / math.sqrt(len(nx)), **kw)


WINDOW = dict(move_window=1, inject_ppc=(1, 1, 1), inject_w=-1.0)


@pytest.mark.parametrize("kw", [
    _box((62, 77, 74), shape_order=3, **WINDOW),
    _box((26, 82, 52), shape_order=2, **WINDOW),
    _box((33, 22, 17), shape_order=2, **WINDOW),
    _box((96, 64, 64), shape_order=2, tile=(48, 0, 0)),
    _box((25, 272), shape_order=3, tile=(0, 272)),
    _box((256, 128), 0.7, shape_order=2, tile=(0, 64), sort_interval=12, chunk=2048),
    _box((42, 116), 0.7, shape_order=2, sort_interval=40),
    # the padded LDS strides of a tile do not grow with its extents alone
    dict(ndim=3, nx=(45, 6, 32), dx=(1.0, 1.0, 0.05), dt=0.014962640041614492, shape_order=2, sort_interval=13,
         accumulator=2),
    dict(ndim=3, nx=(99, 88, 38), dx=(0.21,) * 3, dt=0.036373066958946425, shape_order=3, sort_interval=4,
         accumulator=2),
], ids=lambda kw: "x".join(map(str, kw["nx"])))
def test_boxes_that_have_a_tile_are_taken(pic, kw):
    assert _taken(pic, **kw)


def _draw(r):
    kind = r.choice(["window", "rz", "partial", "long", "plain"])
    dim = 2 if kind == "rz" else r.choice([2, 3])
    nx = tuple(r.randint(2, 140) for _ in range(dim))
    dx = tuple(r.choice([0.05, 0.2, 0.21, 1.0]) for _ in range(dim))
    kw = dict(ndim=dim, nx=nx, dx=dx, dt=r.choice([0.3, 0.95]) / math.sqrt(sum(1 / d ** 2 for d in dx)),
              shape_order=r.randint(1, 3), accumulator=r.choice([0, 0, 2]), chunk=r.choice([0, 0, 256, 2048]))
    asked = [0] * dim
    if kind == "window" or (kind == "rz" and r.random() < 0.5):
        kw.update(WINDOW)
    if kind == "rz":
        kw["geometry"] = 1  # PIC_GEOM_RZ
    if kind in ("partial", "long"):
        kw["sort_interval"] = 1 if kind == "partial" or "move_window" in kw else r.randint(2, 50)
    if kind in ("partial", "long"):
        asked = [r.choice([0, r.randint(1, n), n, 8]) for n in nx]
    if kw["shape_order"] == 1 and r.random() < 0.3:
        kw["deposit"] = 1
    return kw, asked


@pytest.mark.parametrize("seed", range(4))
def test_default_is_taken_where_an_asked_tile_is(pic, seed):
    """Every box that is taken with a small tile asked for on its free axes is
    taken without."""
    r = random.Random(seed)
    both = 0
    for _ in range(1500):
        kw, asked = _draw(r)
        si = kw.get("sort_interval") or 1
        least = []
        for d, n in enumerate(kw["nx"]):
            need = 3 + max(0, math.ceil((si - 1) * kw["dt"] / kw["dx"][d] - 1e-12))
            ok = [t for t in range(need, n) if n % t == 0 or n % t >= need]
            least.append(asked[d] or (ok[0] if ok else n))
        short = dict(kw, tile=tuple(least), sort_interval=si)
        if _taken(pic, **short):
            both += 1
            assert _taken(pic, tile=tuple(asked), **kw), (kw, asked)
    assert both > 500  # (the sweep reaches boxes that are taken)
