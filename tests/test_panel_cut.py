"""How the panel, block and fp32 GEMMs cut their launches, on the CPU: their host functions (tests/panel_stub.cpp) for devices of several sizes."""
import ctypes
import os
import subprocess

import pytest

from paper_2304_04487_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("panel")
    obj = str(tmp / "panel.o")

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return r.stdout

    run([build._hipcc(), "-std=c++17", "-O1", "-fPIC", "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-Wno-unused-result",
         "-I", build.CSRC, "-c", os.path.join(HERE, "panel_stub.cpp"), "-o", obj])
    no_code = [f"-Wl,--defsym={w}=0" for w in run(["nm", "-u", obj]).split() if w.startswith("__hip_fatbin")]

    def open_for(units):                        # a library each: the number of units is asked for once
        out = str(tmp / f"panel_{units}.so")
        run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,--no-undefined", *no_code, "-o", out, obj])
        lib = ctypes.CDLL(out)
        lib.stub_compute_units(units)
        return lib
    return open_for


@pytest.mark.parametrize("units", [256, 128, 64, 32])
def test_every_row_has_its_rstd(library, units):
    """in the split-K form the waves of the first kernel share the rows' rstd: all rows, also of a narrow matrix (few waves)
    with many of them"""
    lib = library(units)
    split = 0
    for d in (512, 768, 1024, 2048, 4096):
        for width in (16, 64, 128, 192, 224, 256, 512, 1040, 2848):
            for rows in [*range(49, 2200, 41), 643, 648, 1152, 1281, 1287, 1664, 1801, 2047, 2048, 3000, 4224]:
                # LM head of a step; gate/up of a step and of a prompt pass; QKV of a prompt pass
                for shape in ((width, d, 1, rows, 0), (width, d, 2, rows, 0), (width, d, 2, min(rows, 2048), 1), (3 * d, d, 1, min(rows, 2048), 1)):
                    missing = lib.stub_rows_without_rstd(*shape)
                    split += missing >= 0
                    assert missing <= 0, (units, shape, missing)
    assert split > 1000


SHAPES = [(d, f) for d, f in ((512, 1408), (4096, 11008), (5120, 13824), (4096, 11088), (1040 * 2, 5632))]


@pytest.mark.parametrize("units", [256, 128, 64, 32])
def test_block_gemm_reads_tiles_that_exist(library, units):
    """every weight and row tile that the block GEMM's workgroups fetch belongs to the matrix and to the pass: ragged last feature blocks and
    last row blocks of QKV, O, gate/up and down"""
    lib = library(units)
    taken, outside = {12: 0, 16: 0}, ctypes.c_int()
    for d, f in SHAPES:
        for rows in range(49, 2049, 13):
            for shape in ((3 * d, d, 1), (d, d, 1), (f, d, 2), (d, f, 1)):
                rt = lib.stub_block_tiles_outside(*shape, rows, ctypes.byref(outside))
                assert outside.value == 0, (units, shape, rows, rt, outside.value)
                if rt:
                    taken[rt] += 1
    assert min(taken.values()) > 50


@pytest.mark.parametrize("at,nw", [(1, 8), (2, 8), (2, 7), (2, 6), (2, 5)])
def test_any_height_of_row_blocks_is_launched(library, at, nw):
    """a cut of a height that some form does not have runs in another one: the finishing kernel would add what the last launch left otherwise"""
    lib = library(256)
    for rt in range(4, 20):
        for rows in (49, 160, 161, 192, 193, 400):
            assert lib.stub_panel_covers(at, nw, 4096, 4096, rows, rt) >= (rows + 15) // 16, (rt, rows)


# us of one launch inside prompt passes on 256 compute units, the forms in turn: ((N, K, tiles per task), rows): panel, blocks of 12, of 16
QKV_7B, QKV_13B, O_13B, GU_7B, GU_13B = (12288, 4096, 1), (15360, 5120, 1), (5120, 5120, 1), (11008, 4096, 2), (13824, 5120, 2)
MEASURED = [
    (GU_7B, 335, 126.2, 128.1, 163.7), (GU_7B, 431, 143.1, 236.4, 164.0), (GU_7B, 847, 247.2, 260.8, 321.5), (GU_7B, 1327, 375.5, 382.7, 482.1),
    (GU_7B, 1536, 425.2, 401.4, 486.5), (GU_7B, 2048, 564.2, 535.9, 513.3), (QKV_7B, 911, 165.8, 156.1, 192.3), (QKV_7B, 1280, 213.9, 276.8, 199.0),
    (QKV_7B, 1679, 281.5, 297.6, 357.1), (QKV_7B, 1920, 319.7, 303.8, 368.4), (QKV_7B, 2048, 331.9, 422.6, 371.6), (GU_13B, 416, 193.4, 291.1, 201.9),
    (GU_13B, 512, 218.8, 294.6, 201.5), (GU_13B, 1103, 453.4, 463.0, 591.2), (GU_13B, 1711, 705.2, 641.7, 787.5), (GU_13B, 1792, 709.4, 781.2, 794.6),
    (GU_13B, 2016, 802.9, 814.7, 833.0), (QKV_13B, 768, 199.4, 186.1, 222.3), (QKV_13B, 847, 229.1, 321.5, 238.9), (QKV_13B, 1024, 258.2, 331.7, 240.4),
    (QKV_13B, 1327, 341.1, 354.8, 436.3), (QKV_13B, 2048, 512.5, 537.5, 473.5), (O_13B, 1664, 173.6, 177.0, 215.7), (O_13B, 2016, 201.1, 316.5, 229.3),
    ((9216, 3072, 1), 1216, 144.4, 204.1, 148.4), ((9216, 3072, 1), 1951, 219.1, 229.1, 281.7), ((8192, 2048, 2), 1024, 105.2, 133.0, 96.4),
]


@pytest.mark.parametrize("shape,rows,panel,b12,b16", MEASURED)
def test_blocks_where_they_are_faster(library, shape, rows, panel, b12, b16):
    """the rule never takes a form that was measured slower than the panel GEMM, and takes one that was 5 % faster"""
    times = {0: panel, 12: b12, 16: b16}
    chosen = times[library(256).stub_block_tiles_outside(*shape, rows, ctypes.byref(ctypes.c_int()))]
    assert chosen <= panel
    assert chosen <= 1.05 * min(times.values())


# us of one fp32 launch: (N, K, epilogue), rows: the kernel with eight rows per wave of before the split; 2, 4, 8 rows per wave now
RESID, SWIGLU, LMHEAD, QKV = 1, 2, 3, 4
MEASURED_F32 = [
    ((384, 128, QKV), 5, 4.6, 2.8, 3.5, 4.2), ((1536, 512, QKV), 16, 7.9, 6.1, 6.0, 6.8), ((2048, 512, SWIGLU), 16, 11.9, 10.2, 8.7, 9.5), ((512, 2048, RESID), 48, 12.0, 11.6, 10.4, 11.1),
    ((3072, 1024, QKV), 9, 10.1, 8.4, 7.9, 9.5), ((3072, 1024, QKV), 48, 23.9, 26.5, 21.2, 21.3), ((4096, 1024, SWIGLU), 48, 51.1, 60.2, 47.5, 45.1), ((1024, 4096, RESID), 5, 12.2, 8.3, 9.2, 11.4),
    ((1024, 4096, RESID), 48, 30.9, 36.0, 30.4, 29.6), ((6144, 2048, QKV), 4, 19.4, 17.4, 15.4, 19.1), ((6144, 2048, QKV), 8, 21.7, 26.9, 21.9, 21.0), ((6144, 2048, QKV), 48, 70.8, 106.5, 88.7, 69.0),
    ((2048, 2048, RESID), 5, 11.5, 8.5, 9.2, 10.8), ((2048, 2048, RESID), 48, 31.7, 39.1, 32.6, 30.8), ((8192, 2048, SWIGLU), 2, 39.0, 27.0, 30.0, 39.0), ((8192, 2048, SWIGLU), 33, 142.0, 203.0, 177.6, 139.7),
    ((8000, 2048, LMHEAD), 33, 116.2, 153.0, 121.1, 113.8), ((12288, 4096, QKV), 5, 60.0, 77.8, 75.0, 60.0), ((12288, 4096, QKV), 48, 272.4, 430.6, 356.9, 269.8),
    ((11008, 4096, SWIGLU), 4, 97.0, 107.0, 86.0, 98.0), ((11008, 4096, SWIGLU), 24, 334.8, 506.5, 500.5, 336.3), ((4096, 11008, RESID), 2, 73.0, 41.0, 48.0, 74.0), ((4096, 11008, RESID), 24, 195.4, 243.7, 215.2, 197.3),
]


@pytest.mark.parametrize("shape,rows,before,two,four,eight", MEASURED_F32)
def test_fp32_rows_per_wave(library, shape, rows, before, two, four, eight):
    """the form taken is no slower than eight rows per wave were, from the smallest models to the widest"""
    assert {2: two, 4: four, 8: eight}[library(256).stub_f32_rows_per_wave(*shape, rows)] <= 1.015 * before


def test_forms_that_the_gpu_tests_are_about(library):
    """on 256 compute units: what tests/test_gpu_tall_panels.py, test_gpu_prompt_blocks.py and test_gpu_f32_kernels.py say that their launches take"""
    lib, outside = library(256), ctypes.c_int()
    for rows in (161, 175, 176, 177, 192):
        assert lib.stub_split_height(*GU_7B, rows, 1) == (rows + 15) // 16, rows
    assert all(lib.stub_split_height(*GU_7B, rows, 1) <= 10 for rows in (160, 193))
    assert all(lib.stub_split_height(*QKV_7B, rows, 0) == (rows + 15) // 16 for rows in (161, 176, 177, 192))       # (steps; see kernels_bf16.hip)
    height = lambda shape, rows: lib.stub_block_tiles_outside(*shape, rows, ctypes.byref(outside))
    assert [height((8192, 2048, 2), rows) for rows in (2047, 2033)] == [16, 16]
    assert [height((6144, 2048, 1), rows) for rows in (1905, 1889)] == [12, 12]
    for shape in ((6336, 2112, 1), (2112, 2112, 1), (2112, 2112, 2)):                       # unsplit: LLMA_BLOCK_ROWS applies
        assert all(lib.stub_split_height(*shape, rows, 1) == 0 for rows in (2047, 1905, 1889, 1500)), shape
    rows_per_wave = lambda shape: [lib.stub_f32_rows_per_wave(*shape, rows) for rows in (2, 3, 4, 5, 12, 17, 33)]
    assert rows_per_wave((6144, 2048, QKV)) == [2, 2, 4, 8, 8, 8, 8]
    assert rows_per_wave((2048, 2048, RESID)) == [2, 2, 2, 2, 8, 8, 8]
    assert rows_per_wave((6002, 2048, SWIGLU)) == [2, 4, 4, 8, 8, 8, 8]
    assert rows_per_wave((2048, 6002, RESID)) == [2, 2, 4, 8, 8, 8, 8]
    assert rows_per_wave((8000, 2048, LMHEAD)) == [2, 4, 4, 8, 8, 8, 8]
