"""Registers of the built kernels (host only: read from the code objects in
liblcsm.so).  A launch that is bound by memory round trips lives on the waves
that fit a SIMD, 512 registers a lane shared among them, so a kernel whose
register use grows by accident loses speed that no parity test sees."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2410_12982_amd", "liblcsm.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of every offload bundle in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


@pytest.fixture(scope="module")
def vgprs(tmp_path_factory):
    """VGPRs of every kernel by mangled name."""
    if not shutil.which(READELF):
        pytest.skip("llvm-readelf is not installed")
    d = tmp_path_factory.mktemp("co")
    out = {}
    with open(LIB, "rb") as f:
        blob = f.read()
    for k, co in enumerate(_code_objects(blob)):
        path = d / f"{k}.co"
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True,
                               text=True).stdout
        for name, count in re.findall(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_count:\s+(\d+)", notes, re.S):
            out[name] = int(count)
    assert out
    return out


@pytest.mark.parametrize("U,K,waves", [(0, 8, 8), (1, 8, 8), (2, 1, 8), (8, 1, 8), (16, 1, 5),
                                       (32, 1, 3)])
def test_single_position_chain_keeps_its_waves(vgprs, U, K, waves):
    """k_chain_fused<U, K>: U = 0 and 1 for contexts of many layers, U up to 32
    for one layer."""
    got = [v for n, v in vgprs.items() if f"k_chain_fusedILi{U}ELi{K}E" in n]
    assert len(got) == 1
    assert got[0] <= 512 // waves


@pytest.mark.parametrize("N", [128, 256, 1024])
def test_row_panel_tile_keeps_two_workgroups(vgprs, N):
    """Every form of k_fft_tile<N> (whole and ragged panels, with and without the
    red cell): at most 128 registers, the limit of four waves per SIMD, which at
    2U = 1024 are two workgroups of 512 threads per compute unit."""
    got = [v for n, v in vgprs.items() if f"k_fft_tileILi{N}ELb0E" in n or f"k_fft_tileILi{N}ELb1E" in n]
    assert len(got) >= 4
    assert max(got) <= 128


def test_profile_grouping_knows_every_step_and_tile_kernel(vgprs):
    """The profile summaries group dispatches by kernel name: every kernel that a
    teacher-forced generation launches is one of their keys, and every step form
    is among the dispatches of its launch."""
    import bench
    if not shutil.which("c++filt"):
        pytest.skip("c++filt is not installed")
    names = subprocess.run(["c++filt", *vgprs], check=True, capture_output=True, text=True).stdout.split("\n")
    short = [bench.short_name(n) for n in names if n]
    path = ("k_step_fused", "k_fft_tile", "k_fft_coltile", "k_cm_", "k_rows_to_cols", "k_cols_to_rows",
            "k_fft_rows_inv", "k_fft_rows_fwd", "k_fft_mid_tile")
    timed = [n for n in short if n.startswith(path)]
    assert len(timed) > 50
    assert [n for n in timed if bench.kernel_key(n) is None] == []
    for U in (1, 2, 4, 8, 16, 32, 64):
        keep = bench.group_kernels("fused", U)
        assert len([n for n in timed if keep(n)]) == 2  # destination whole and clipped
