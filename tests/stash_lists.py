"""What a count pass left in the workspace: the lengths of its lists and the
words of the stash header (counter block of the query workspace)."""
import os
import re

import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _layout():
    with open(os.path.join(ROOT, "paper_cs_0608108_amd", "csrc", "sphidx_internal.h")) as f:
        text = f.read()
    return {k: int(re.search(rf"#define SPHIDX_{k}\s+(\d+)", text).group(1)) for k in ("NQUEUE", "QSTRIDE", "NQSETS")}


NAMES = ("long", "fallback", "walk", "header", "extra", "long_expected", "items", "big")


def lists(buf):
    """{name: length} of the lists, `kept` (the header says that rows were
    kept) and `tiles` (counted by tiles, rows kept)."""
    lay = _layout()
    torch.cuda.synchronize()
    off = buf._ws - buf.workspace.data_ptr()
    words = lay["NQUEUE"] * lay["QSTRIDE"] * lay["NQSETS"] + len(NAMES) * lay["QSTRIDE"]
    w = buf.workspace[off:off + 4 * words].view(torch.int32).cpu().numpy()
    w = w[lay["NQUEUE"] * lay["QSTRIDE"] * lay["NQSETS"]:].reshape(len(NAMES), lay["QSTRIDE"])
    out = {n: int(w[i, 0]) for i, n in enumerate(NAMES) if n != "header"}
    h = w[NAMES.index("header")]
    out["kept"], out["tiles"] = bool(h[0]), bool(h[4])
    return out
