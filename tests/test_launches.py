"""What the C calls launch, recorded under a stand-in for the HIP runtime
(launch_recorder.c, no GPU): a call whose grids HIP would refuse launches
nothing and says so."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2609_27373_amd import wise

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests")

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="no C compiler")


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if not os.path.exists(wise.LIB_PATH):
        from paper_2609_27373_amd import build
        build.build()
    exe = tmp_path_factory.mktemp("rec") / "recorder"
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "launch_recorder.c"), "-o", str(exe), wise.LIB_PATH,
                    f"-Wl,-rpath,{os.path.dirname(wise.LIB_PATH)}"], check=True, capture_output=True, text=True)

    def record(entry, batch, heads, n, d, block, option=1, kv_heads=1):
        """([(verdict, kernel, grid x, y, z, threads, dynamic LDS, template arguments)], status) of one call."""
        line = f"{entry} {batch} {heads} {kv_heads} {n} {d} {block} {option}\n"
        out = subprocess.run([str(exe)], input=line, capture_output=True, text=True, timeout=60, check=True).stdout.split("\n")
        launches = []
        for ln in out:
            f = ln.split()
            if f and f[0] in ("launch", "refused"):
                launches.append((f[0], re.search(r"\d+([a-z]+(?:_[a-z0-9]+)*_kernel)", f[1]).group(1), *map(int, f[2:]),
                                 tuple(int(x) for x in re.findall(r"Li(\d+)E", f[1]))))
        return launches, int(out[-2].split()[1])

    return record


WISE_ERR_HIP = 6


def test_recorder(recorder):
    launches, status = recorder("dense", 1, 32, 4096, 128, 64, kv_heads=32)
    assert status == 0 and launches == [("launch", "dense_attn_kernel", 512, 1, 1, 512, 0, (128, 8, 0))]


# 2^26 rows: 64 threads each are more than a grid holds
@pytest.mark.parametrize("entry", ["select", "step", "support"])
@pytest.mark.parametrize("heads,nb", [(1 << 21, 32), (1 << 26, 1)])
@pytest.mark.parametrize("order", [0, 1])
def test_refused_rows_launch_nothing(recorder, entry, heads, nb, order):
    launches, status = recorder(entry, 1, heads, 64 * nb, 64, 64, order)
    assert status == WISE_ERR_HIP
    assert all(verdict == "refused" for verdict, *_ in launches), launches


@pytest.mark.parametrize("heads,nb", [(2147483647, 1), (1 << 30, 1)])
def test_refused_union_launches_nothing(recorder, heads, nb):
    launches, status = recorder("masks", 1, heads, 64 * nb, 64, 64)
    assert status == WISE_ERR_HIP
    assert all(verdict == "refused" for verdict, *_ in launches), launches


# Up to 16777215 heads and 2^26 - 1 rows were accepted when each head's order had a 256-thread group.
@pytest.mark.parametrize("heads,nb", [(1 << 22, 1), (6000000, 2), (16777215, 1), (16777215, 3), ((1 << 21) - 1, 32), (500000, 90), (1 << 17, 129)])
@pytest.mark.parametrize("entry", ["select", "masks"])
def test_many_heads_are_accepted(recorder, entry, heads, nb):
    launches, status = recorder(entry, 1, heads, 64 * nb, 64, 64)
    assert status == 0
    assert all(verdict == "launch" for verdict, *_ in launches), launches


@pytest.mark.parametrize("heads,nb", [(100000, 2), (8192, 16), (1000, 1), (512, 1), (513, 1), (1600, 42), (1600, 43), (2000, 64), (2000, 65), (9, 128),
                                      (9, 129), (2, 1024)])
def test_csr_groups_hold_whole_heads(recorder, heads, nb):
    """128 rows of a head, or as many heads as 128 rows allow, once every head cannot have one of 512 groups."""
    launches, _ = recorder("masks", 1, heads, 64 * nb, 64, 64)
    (x, y), = [(f[2], f[3]) for f in launches if f[1] == "csr_kernel"]
    per = min(max(1, 128 // nb), -(-heads // 512))
    assert (x, y) == (-(-heads // per), -(-nb // 128))


@pytest.mark.parametrize("heads,nb,scan", [(1024, 128, False), (8192, 128, False), (8128, 129, False), (8200, 129, True), (1 << 22, 1, True)])
def test_scan_only_past_the_sums(recorder, heads, nb, scan):
    launches, status = recorder("masks", 1, heads, 64 * nb, 64, 64)
    assert status == 0 and [f[1] for f in launches] == ["union_rows_kernel"] + ["scan_kernel"] * scan + ["csr_kernel"]


# One row a work-group of 64- and 128-key blocks: two tiles in LDS for 128-key blocks and in small grids, and
# at d 96 four groups a CU in grids below 2048 rows
@pytest.mark.parametrize("d,block,heads,nb,bufs,lds", [
    (64, 64, 16, 64, 2, 32768), (64, 64, 17, 64, 1, 16384), (96, 64, 20, 64, 2, 49152), (96, 64, 21, 64, 1, 40960), (96, 64, 31, 64, 1, 40960),
    (96, 64, 32, 64, 1, 24576), (96, 64, 33, 64, 1, 24576), (128, 64, 12, 64, 2, 65536), (128, 64, 13, 64, 1, 32768),
    (64, 128, 2, 4, 2, 32768), (96, 128, 200, 32, 2, 49152), (128, 128, 64, 128, 2, 65536)])
def test_late_rows_route(recorder, d, block, heads, nb, bufs, lds):
    (launch,), status = recorder("sparse", 1, heads, nb * block, d, block)
    assert status == 0 and launch[0] == "launch" and launch[1] == "sparse_attn_kernel"
    assert launch[5:] == (block * 2, lds, (d, block // 32, bufs))
