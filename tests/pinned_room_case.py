"""One process of test_gpu_direct.py's test of pinned memory: dumps under a
small pinned budget (MICKPT_PINNED_BUDGET, read when the library is first
used) of states that are mostly zero behind a dense start, by the form given;
every image must be pinned and right."""
import os
import sys
import tempfile

import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2502_16631_amd import mickpt as mk  # noqa: E402

MIB = 1 << 20


def main(form):
    ctx = mk.ckpt_ctx_create(0, 6 << 30)
    size, images = {"long": (4 << 30, 2), "many": (1 << 30, 20), "graph": (1 << 30, 12), "short": (18 * MIB, 150),
                    "file": (1 << 30, 6)}[form]
    t = torch.zeros(size, dtype=torch.uint8, device="cuda")
    dense = t[: size // 16]
    table, kept = [(1, t)], []
    opts = mk.make_opts(flags=mk.OPT_GRAPH if form == "graph" else 0)
    for i in range(images):
        dense.random_(1, 256)
        torch.cuda.synchronize()
        if form == "file":
            with tempfile.NamedTemporaryFile() as f:
                rc, img, res = mk.ckpt_dump_file(ctx, table, f.name, keep_image=True)
        else:
            rc, img, res = mk.ckpt_dump(ctx, table, opts=opts)
        assert rc == 0
        v = torch.from_numpy(img.view())
        print(form, i, img.nbytes(), v.is_pinned(), flush=True)
        assert v.is_pinned(), "image %d of %d bytes is not pinned" % (i, img.nbytes())
        assert res.n_payload == dense.numel()
        assert torch.equal(v[-dense.numel():].cuda(), dense)
        kept.append((img, v))
    to = [(1, torch.full_like(t, 7))]
    assert mk.ckpt_restore(ctx, kept[-1][0], to)[0] == 0
    torch.cuda.synchronize()
    assert torch.equal(to[0][1], t)
    print("all pinned")


if __name__ == "__main__":
    main(sys.argv[1])
