"""Register, scratch and occupancy facts of the compiled gfx950 kernels.

build() keeps the compiler's per-kernel resource report of every kernel
source (hipcc -Rpass-analysis=kernel-resource-usage) beside the objects.
These tests read it and hold the kernels to the budget their design assumes:
no per-subset or batch instance spills to scratch except the one held to
three waves on purpose, the launched series kernels stay free of scratch but
for the largest order, and the instances that carry the N = 50 benchmark keep
the waves per SIMD that their timings were taken at.  CPU only; skipped when
no build has left the report."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2010_15595_amd", "_build")
SOURCES = ["charpoly_l44.hip", "charpoly_l84.hip", "charpoly_l88.hip", "lhaf_kernels.hip", "lhaf_lds.hip",
           "sampler_kernels.hip"]

# <P, Q, MR, MC, type, TEAM, O> from the Itanium-mangled instance name
_TILE = re.compile(r"_ZN3gbs(\d+)(charpoly_kernel|charpoly_batch_kernel)ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E"
                   r"15HIP_vector_typeI([df])Lj2EELi(\d+)ELi(\d+)E")
_SERIES = re.compile(r"_ZN3gbs\d+(series_kernel|series_batch_kernel)ILi(\d+)E15HIP_vector_typeI([df])Lj2EE")


def _report():
    files = [os.path.join(BUILD, s + ".resources.txt") for s in SOURCES]
    if not all(os.path.exists(f) for f in files):
        pytest.skip("no resource report: run __graft_entry__.build() first")
    kernels = {}
    for path in files:
        cur = None
        with open(path) as f:
            for line in f:
                m = re.search(r"remark: Function Name: (\S+)", line)
                if m:
                    cur = kernels.setdefault(m.group(1), {})
                    continue
                m = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\S+) \[-Rpass", line)
                if m and cur is not None:
                    cur[m.group(1).strip()] = m.group(2)
    return kernels


def _tiles(kernels):
    out = {}
    for name, r in kernels.items():
        m = _TILE.match(name)
        if m:
            kind, P, Q, MR, MC, t, team, O = m.group(2), *map(int, m.group(3, 4, 5, 6)), m.group(7), \
                *map(int, m.group(8, 9))
            out[(kind, P, Q, MR, MC, "f64" if t == "d" else "f32", team, O)] = r
    return out


@pytest.fixture(scope="module")
def kernels():
    return _report()


def test_report_covers_every_kernel_source(kernels):
    # every instance the parser reads: 156 per-subset and 104 batch tiles
    # (both precisions), the series kernels of every order in both precisions
    tiles = _tiles(kernels)
    assert sum(k[0] == "charpoly_kernel" for k in tiles) == 156
    assert sum(k[0] == "charpoly_batch_kernel" for k in tiles) == 104
    assert sum(bool(_SERIES.match(n)) for n in kernels) == 4 * 32
    assert all("ScratchSize" in r and "Occupancy" in r for r in kernels.values())


def test_tile_instances_stay_out_of_scratch(kernels):
    """Every per-subset and batch tile instance keeps its values in registers,
    except the FP64 one-team 8 x 4 3 x 6 tile at offset 0, which is held to
    three waves per SIMD and spills a few registers by design."""
    held = ("charpoly_kernel", 8, 4, 3, 6, "f64", 64, 0)
    spilled = {}
    for key, r in _tiles(kernels).items():
        if int(r["ScratchSize"]) > 0:
            spilled[key] = int(r["ScratchSize"])
    assert set(spilled) == {held}, spilled
    assert spilled[held] <= 16
    assert int(_tiles(kernels)[held]["Occupancy"]) == 3


def test_series_kernels_of_launched_orders_stay_out_of_scratch(kernels):
    """Single evaluations launch the series kernel for n = 1..32 (only the
    FP64 order-32 instance, N = 63 and 64, spills); batch plans stop at
    N = 56 (n <= 28), so their launched orders never spill."""
    spills = {}
    for name, r in kernels.items():
        m = _SERIES.match(name)
        if m and int(r["ScratchSize"]) > 0:
            spills[(m.group(1), int(m.group(2)), m.group(3))] = int(r["ScratchSize"])
    singles = {k for k in spills if k[0] == "series_kernel"}
    assert singles <= {("series_kernel", 32, "d")}, spills
    assert not [k for k in spills if k[0] == "series_batch_kernel" and k[1] <= 28], spills


@pytest.mark.parametrize("key, waves", [
    (("charpoly_kernel", 8, 4, 4, 7, "f64", 64, 2), 2),   # s = 13 of N = 50
    (("charpoly_kernel", 8, 4, 4, 7, "f64", 64, 0), 2),   # column-swap map
    (("charpoly_kernel", 8, 4, 4, 8, "f64", 64, 0), 2),   # column-swap map
    (("charpoly_kernel", 8, 4, 4, 8, "f64", 64, 2), 2),
    (("charpoly_kernel", 8, 4, 3, 6, "f64", 64, 2), 3),
    (("charpoly_kernel", 8, 4, 3, 5, "f64", 64, 0), 3),
    (("charpoly_kernel", 8, 8, 4, 4, "f64", 64, 4), 3),   # s = 14 of N = 50
    (("charpoly_kernel", 8, 8, 5, 5, "f64", 64, 6), 2),
    (("charpoly_kernel", 8, 4, 4, 8, "f32", 32, 0), 2),   # FP32 twin of the 4 x 8 tile
])
def test_benchmark_instances_keep_their_occupancy(kernels, key, waves):
    r = _tiles(kernels)[key]
    assert int(r["Occupancy"]) == waves, (key, r)
    assert int(r["VGPRs"]) + int(r["AGPRs"]) <= 512 // waves


def test_subset_tree_kernels_stay_out_of_scratch():
    """Every subset-tree instance keeps its series in registers."""
    path = os.path.join(BUILD, "lhaf_kernels.hip.resources.txt")
    if not os.path.exists(path):
        pytest.skip("no resource report: run __graft_entry__.build() first")
    with open(path) as f:
        text = f.read()
    names = re.findall(r"Function Name: (\S+)", text)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", text)]
    assert len(names) == len(scratch)
    tree = {}
    for name, x in zip(names, scratch):
        m = re.search(r"tree_(sub|elim)_kernelILi(\d+)", name)
        if m:
            tree.setdefault(m.group(1), set()).add(int(m.group(2)))
            assert x == 0, name
        if "tree_top_elim" in name:
            assert x == 0, name
    assert tree["sub"] == set(range(1, 29)) and tree["elim"] == set(range(6, 29))


def test_double_double_tree_kernels_stay_out_of_scratch():
    path = os.path.join(BUILD, "lhaf_lds.hip.resources.txt")
    if not os.path.exists(path):
        pytest.skip("no resource report: run __graft_entry__.build() first")
    with open(path) as f:
        text = f.read()
    names = re.findall(r"Function Name: (\S+)", text)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", text)]
    found = [x for name, x in zip(names, scratch) if "tree_" in name]
    assert len(found) == 7 and not any(found)
