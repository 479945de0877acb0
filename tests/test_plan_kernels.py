"""fftsplit_plan_kernels: what it reports is what the launch code dispatches on
(one field of the plan), and the shapes of the GPU tests run the kernels that
those tests are about.  No GPU needed."""
import ctypes
import os
import re
import subprocess

import pytest

import paper_2003_12621_amd as fs

from test_abi_host import HEADER, ROOT
from test_gpu_contract_split import CASES, _tile
from test_gpu_direct_split import CASES as DIRECT_CASES
from test_gpu_oaa_strip import CASES as STRIP_CASES


def plan(shape, tile=0):
    return fs.Plan(*shape, tile=tile, mode="oaa" if tile == shape[5] else "os", arch="gfx950")


@pytest.mark.parametrize("shape,tile,kernel", CASES)
def test_contraction_tiles(shape, tile, kernel):
    assert _tile(plan(shape, tile)) == kernel


def test_every_tile_has_a_case():
    text = open(os.path.join(ROOT, "paper_2003_12621_amd", "csrc", "fftsplit_internal.hpp")).read()
    table = text[text.index("kSplitTileShapes[] ="):]
    tiles = re.findall(r"\{(\d+), (\d+), (\d+)\}", table[:table.index(";")])
    assert {tuple(map(int, t)) for t in tiles[1:]} == {kernel for _, _, kernel in CASES}


@pytest.mark.parametrize("shape", DIRECT_CASES)
def test_direct_blocks(shape):
    k = plan(shape).kernels
    assert k.direct_split and k.direct_block_w in (8, 16, 32, 64)


def test_all_direct_block_widths_have_a_case():
    assert {plan(s).kernels.direct_block_w for s in DIRECT_CASES} == {8, 16, 32, 64}


def test_fp32_contraction_is_reported_as_such(monkeypatch):
    """Patches padded to an odd multiple of 32, and the environment variables."""
    def fields(p):
        k, i = p.kernels, p.info
        return (k.contract_split, k.contract_part_products, (k.contract_tile_m, k.contract_tile_n, k.contract_stage_k,
                k.contract_prefetch, k.contract_real_products) == (i.contract_tile_m, i.contract_tile_n,
                                                                   i.contract_stage_k, i.contract_prefetch,
                                                                   i.contract_real_products))
    assert fields(plan((32, 512, 14, 14, 512, 3), 14)) == (0, 1, True)
    headline = (16, 256, 56, 56, 256, 5)
    k = plan(headline, 28).kernels
    assert (k.contract_split, k.contract_tile_m, k.contract_tile_n) == (1, 256, 64)
    assert (k.contract_real_products, k.contract_part_products) == (4, 6)
    monkeypatch.setenv("FFTSPLIT_CONTRACT_SPLIT", "0")
    monkeypatch.setenv("FFTSPLIT_DIRECT_SPLIT", "0")
    assert fields(plan(headline, 28)) == (0, 1, True)
    assert plan(headline, 28).kernels.direct_split == 0
    monkeypatch.delenv("FFTSPLIT_CONTRACT_SPLIT")
    monkeypatch.setenv("FFTSPLIT_CONTRACT_TILE", "g4:64x64x32")
    assert fields(plan(headline, 28)) == (0, 1, True)


@pytest.mark.parametrize("value,split", [("", 1), ("0", 1), ("7", 1), ("1", 0), ("3", 0)])
def test_prefetch_variable_that_asks_for_nothing(value, split, monkeypatch):
    monkeypatch.setenv("FFTSPLIT_CONTRACT_PREFETCH", value)
    assert plan((16, 256, 56, 56, 256, 5), 28).kernels.contract_split == split


@pytest.mark.parametrize("shape,strip", STRIP_CASES)
def test_oaaconv_strips(shape, strip):
    k = plan(shape, shape[5]).kernels
    assert (k.oaaconv_strip_rows, k.oaaconv_strip_images) == strip


@pytest.mark.parametrize("k,widest", [(3, 1167), (5, 675), (7, 469)])
def test_oaaconv_strip_limit(k, widest):
    """Four patch rows of an image fit a strip up to this many columns."""
    rows = [plan((1, 1, 8 * k, w, 2, k), k).kernels.oaaconv_strip_rows for w in range(8, widest + 200, 3)]
    rows += [plan((1, 1, 8 * k, w, 2, k), k).kernels.oaaconv_strip_rows for w in (widest, widest + 1)]
    assert [bool(r) for r in rows] == [w <= widest for w in [*range(8, widest + 200, 3), widest, widest + 1]]


def test_null_arguments():
    assert fs.lib().fftsplit_plan_kernels(None, ctypes.byref(fs.PlanKernels())) == fs.ERROR_INVALID_VALUE
    assert fs.lib().fftsplit_plan_kernels(plan((1, 3, 32, 32, 16, 3), 6)._h, None) == fs.ERROR_INVALID_VALUE


def test_struct_layout_matches_header(tmp_path):
    names = [f for f, _ in fs.PlanKernels._fields_]
    src = tmp_path / "layout.c"
    src.write_text(f'#include <stddef.h>\n#include <stdio.h>\n#include "{HEADER}"\nint main(void) {{\n'
                   'printf("%zu", sizeof(fftsplit_plan_kernels_t));\n'
                   + "".join(f'printf(" %zu", offsetof(fftsplit_plan_kernels_t, {f}));\n' for f in names)
                   + "return 0;\n}\n")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-x", "c", "-std=c11", "-I", "/opt/rocm/include", "-D__HIP_PLATFORM_AMD__", str(src),
                    "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert [int(v) for v in out] == [ctypes.sizeof(fs.PlanKernels)] + [getattr(fs.PlanKernels, f).offset for f in names]
