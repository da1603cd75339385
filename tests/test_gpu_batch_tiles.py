"""Batched products with two tiles: every assignment of molecules to a pair (all
to the second, some to each, all to the first) and a pair that is out of range
give the results of the contexts alone, as with one tile.  The pairs are put into
a tile table that a second process loads."""
import glob
import json
import os
import re
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import json, sys
import torch, synth
import paper_2512_16677_amd as q
mode = sys.argv[1]
mols = synth.molecule_batch(n_mol=7, seed=11)
err = {}
for n in (4, 5, 6, 7):
    ctxs = [q.Context.from_system(m, mode=mode, points_on_device=True) for m in mols[:n]]
    ws = [torch.from_numpy(synth.adjoint_weights(m, seed=5)).cuda() for m in mols[:n]]
    b = q.Batch(ctxs)
    b.run(ws=ws)
    outs, grads = b.run(ws=ws)
    torch.cuda.synchronize()
    worst = 0.0
    for c, o, g, w in zip(ctxs, outs, grads, ws):
        ref = {"mo": c.get_mo_vgl(), **c.adjoint(w)}
        for k, v in ref.items():
            got = o if k == "mo" else g[k]
            worst = max(worst, float((got.reshape(v.shape) - v).abs().max() / v.abs().max()))
    err[n] = worst
    b.close()
print("ERR " + json.dumps(err), flush=True)
"""


def child(mode, table):
    r = subprocess.run([sys.executable, "-c", CHILD, mode], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env={**os.environ, "QMK_TUNE_CACHE": str(table), "PYTHONPATH": ROOT})
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(re.search(r"ERR (.*)", r.stdout).group(1))


# two tiles of the mode's table; FP64 as in the batch tests (another split of the
# sums over points than alone), BF16x3 products are sums of FP32 terms
@pytest.mark.parametrize("mode,t0,t1,tol", [("fp64", 0, 7, 1e-12), ("mixed_bf16x3", 6, 16, 1e-5)])
def test_pairs_of_tiles(mode, t0, t1, tol, tmp_path):
    table = tmp_path / "tiles.json"
    assert max(child(mode, table).values()) <= tol
    tiles = json.loads(table.read_text())
    ratio = {5: 1, 6: 64, 7: 2047}
    bad = t0 | 201 << 8 | 64 << 16
    forced = {}
    shipped = set()
    for f in glob.glob(os.path.join(ROOT, "paper_2512_16677_amd", "*.json")):
        with open(f) as h:
            shipped |= set(json.load(h))
    for key in set(tiles) - shipped:
        m = re.search(r"/batch/.*/n(\d+)/", key)
        n = int(m.group(1)) if m else 0
        if n:
            forced[key] = bad if n == 4 else t0 | (t1 + 1) << 8 | ratio[n] << 16
    assert len(forced) == 12  # three products of four batches
    table.write_text(json.dumps({**tiles, **forced}, indent=1))
    assert max(child(mode, table).values()) <= tol
    after = json.loads(table.read_text())
    for key, code in forced.items():
        assert (after[key] == code) == (code != bad)
