"""Calls are ordered after the work that the caller's stream holds: pending
work on the given stream, and for the null stream on streams that
synchronize with it."""
import ctypes
import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2502_16631_amd import mickpt as mk  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = mk.ckpt_ctx_create(0, 1 << 30)
    yield c
    mk.ckpt_ctx_destroy(c)


@pytest.fixture(scope="module")
def blocking_stream():
    """A stream that synchronizes with the null stream (torch's do not)."""
    hip = ctypes.CDLL("libamdhip64.so")
    h = ctypes.c_void_p()
    torch.zeros(1, device="cuda")
    assert hip.hipStreamCreate(ctypes.byref(h)) == 0
    yield torch.cuda.ExternalStream(h.value)
    torch.cuda.synchronize()
    hip.hipStreamDestroy(h)


BIG = {}


def pending(stream, table, value):
    """60-90 ms of copies on the stream, then value in every allocation."""
    if not BIG:
        BIG["src"] = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
        BIG["dst"] = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(160):
            BIG["dst"].copy_(BIG["src"], non_blocking=True)
        for _, t in table:
            t.fill_(value)
    assert not stream.query()   # still to come


@pytest.mark.parametrize("where", ["side", "default", "blocking"])
@pytest.mark.parametrize("mib", [1, 24, 160])
def test_calls_wait_for_pending_work(ctx, blocking_stream, where, mib):
    """Dumps (plain, short and long, into the caller's buffer, delta) see what
    pending work writes, and a restore is not overwritten by it."""
    stream = {"side": torch.cuda.Stream(), "default": torch.cuda.default_stream(), "blocking": blocking_stream}[where]
    arg = stream if where == "side" else None
    table = [(i, torch.full((mib << 19,), 1, dtype=torch.uint8, device="cuda")) for i in range(2)]
    tables = 64 + (32 * 2 + 5 * (mib << 4) + 15) // 16 * 16

    def payload(v):
        return v[tables:]

    pending(stream, table, 2)
    rc, img, _ = mk.ckpt_dump(ctx, table, stream=arg)
    assert rc == 0 and (payload(img.view()) == 2).all()
    pending(stream, table, 3)
    rc, delta, res = mk.ckpt_dump(ctx, table, prev=img, stream=arg)
    assert rc == 0 and res.n_data == res.n_chunks and (payload(delta.view()) == 3).all()
    if mib < 160:
        out = torch.empty((mib << 20) + (1 << 20), dtype=torch.uint8, pin_memory=True).numpy()
        pending(stream, table, 4)
        rc, n, _ = mk.ckpt_dump_into(ctx, table, out, stream=arg)
        assert rc == 0 and (payload(out[:n]) == 4).all()
    for call in (lambda: mk.ckpt_restore(ctx, img, table, stream=arg),
                 lambda: mk.ckpt_restore_some(ctx, img, table, stream=arg)):
        pending(stream, table, 5)
        assert call()[0] == 0
        torch.cuda.synchronize()
        assert all((t == 2).all() for _, t in table)
    pending(stream, table, 2)
    rc, _ = mk.ckpt_restore(ctx, delta, table, stream=arg)   # a full rewrite: no chunk is checked against the base
    assert rc == 0
    torch.cuda.synchronize()
    assert all((t == 3).all() for _, t in table)
    assert np.array_equal(img.view()[:8], delta.view()[:8])
    img.free()
    delta.free()
