"""The shipped tile table: every entry names tiles that are on offer, and the sizes
of the benchmark workloads have entries made since the last tile was added to the
lists (a size that is found there is never timed again)."""
import json
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2512_16677_amd")


def table():
    with open(os.path.join(PKG, "tiles_gfx950.json")) as f:
        return json.load(f)


def offered(source, macro):
    with open(os.path.join(PKG, "csrc", source)) as f:
        text = f.read()
    body = re.search(r"#define " + macro + r"\(X\)((?:.*\\\n)*.*\n)", text).group(1)
    return [int(i) for i in re.findall(r"X\((\d+),", body)]


def test_entries_name_tiles_on_offer():
    plain = offered("gemm_impl.h", "QMK_TILE_LIST")
    jastrow = offered("jastrow_product.hip", "QMK_JAS_TILES")
    assert plain == list(range(len(plain))) and jastrow == list(range(len(jastrow)))
    for key, code in table().items():
        assert code >= 0, key
        if "/k4/" in key:
            assert code in jastrow, key
        elif "/batch/" in key:
            tiles = [code & 255] + ([((code >> 8) & 255) - 1] if code >= 256 else [])
            assert "/p3/" in key or all(t in plain for t in tiles), key
        elif "/p3/" not in key:
            assert code in plain, key


def test_benchmark_workloads_have_entries_of_the_present_list():
    t = table()
    for p in (0, 1):
        # 218 occupied orbitals: 224 columns on the 112-wide tiles, 256 on 128-wide ones
        assert t[f"gfx950/k3/p{p}/w0/o0/1000000x218x1114/b1"] in (14, 15)
    assert t["gfx950/k0/p0/w0/o0/1280x25x25"] in (12, 13)  # few workgroups on larger tiles
    assert "gfx950/k4/p0/w5/o0/80x280x280/b512/f" in t
    batches = [code for key, code in t.items() if "/batch/" in key and "/n96/" in key]
    assert len(batches) == 9 and any(code >= 256 for code in batches)
