"""The sizes that launches and workspaces are planned with, on the CPU: a small
program linked with the library answers queries (launch_rules.cpp)."""
import os
import shutil
import subprocess

import pytest

import paper_2603_07038_amd as etm
from paper_2603_07038_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))

pytestmark = pytest.mark.skipif(not shutil.which(B.HIPCC) and not os.path.exists(B.HIPCC),
                                reason="hipcc not available")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    etm.load()  # (built)
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    r = subprocess.run([B.HIPCC] + [f for f in B.FLAGS if f != "-O3"] + ["-O1", "-x", "hip",
                       os.path.join(HERE, "launch_rules.cpp"), "-x", "none", B.LIB, "-Wl,-rpath," + B.HERE, "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]

    def query(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        out = r.stdout.splitlines()
        assert len(out) == len(lines) and not any(x.startswith("error") for x in out), r.stdout
        return [[int(v) for v in x.split()] for x in out]
    return query


# Long meshes of few planes have more operator tiles (31 x 7 nodes) than blocks
# of 64 x 4 nodes; the last two are ordinary ones.
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
def test_solver_partials_hold_every_block(ask, precision):
    shapes = [(32800, 7, 1), (63999, 3, 1), (100000, 7, 1), (65000, 7, 2), (7, 60000, 1), (64, 70, 30000), (31, 7, 1),
              (256, 256, 64)]
    for shape, (rows, fp32, fp64) in zip(shapes, ask(["partials %d %d %d %d" % (precision, *s) for s in shapes])):
        assert rows >= max(fp32, fp64), (shape, rows, fp32, fp64)


# An FP64 block is 256 nodes of a plane: 32 x 8, or 64 x 4 where that takes at
# least a fifth fewer blocks and the launch has more of them than CUs.
def test_fp64_tiles_do_not_idle_on_few_rows(ask):
    shapes = [(nx, ny, nz) for nx in (1, 30, 31, 32, 63, 64, 96, 500, 4000) for ny in (1, 2, 3, 4, 7, 8, 11, 12, 15, 16, 63, 255)
              for nz in (1, 60, 400)]
    for (nx, ny, nz), (tx, ty, kc) in zip(shapes, ask(["tiles %d %d %d %d" % (etm.ETM_PREC_FP64, *s) for s in shapes])):
        tile, flat = -(-(nx + 1) // 32) * -(-(ny + 1) // 8), -(-(nx + 1) // 64) * -(-(ny + 1) // 4)
        want = flat if 5 * flat <= 4 * tile and tile * (nz + 1) > 256 else tile
        assert kc == nz + 1 and tx * ty == want, (nx, ny, nz, tx, ty)


# A mixed plan takes tiles of 64 x 4 nodes when a step's 85 bytes per node (rows
# padded to 16) exceed 256 MB and the tiles pad the plane by at most 30 %, and
# runs of 248 nodes of the plane otherwise: either side of both lines.
def test_mixed_form_switches_where_a_step_streams(ask):
    shapes = [(254, 188, 64), (254, 189, 64), (254, 190, 64), (255, 188, 64), (255, 190, 64), (256, 190, 64), (129, 190, 150),
              (127, 190, 150), (207, 255, 64), (191, 255, 64), (61, 61, 38), (1023, 255, 12), (1024, 1024, 128)]
    got = ask(["tiles %d %d %d %d" % (etm.ETM_PREC_MIXED, *s) for s in shapes])
    forms = []
    for (nx, ny, nz), (tx, ty, kc) in zip(shapes, got):
        nodes = -(-(nx + 1) // 16) * 16 * (ny + 1) * (nz + 1)
        bx, by = -(-(nx + 1) // 64), -(-(ny + 1) // 4)
        tiles = nodes * 85 > 1 << 28 and bx * by * 256 * 10 <= (nx + 1) * (ny + 1) * 13
        want = (bx, by) if tiles else (-(-(nx + 1) * (ny + 1) // 248), 1)
        assert (tx, ty) == want and kc == nz + 1, (nx, ny, nz, tx, ty)
        forms.append(tiles)
    assert forms[:3] == [False, True, True] and not forms[6] and forms[7]


def hex8_chunk(nx, ny, nz, resident):
    """Fewest generations of resident blocks times planes per block, the longest chunk on a tie."""
    tiles = -(-(nx + 1) // 31) * -(-(ny + 1) // 7)
    rows = max(1024, -(-(nx + 1) // 64) * -(-(ny + 1) // 4) * (nz + 1))
    best, least = nz + 1, None
    for kc in range(nz + 1, 1, -1):
        blocks = tiles * -(-(nz + 1) // kc)
        if blocks > rows and kc <= nz:
            break
        cost = -(-blocks // resident) * (kc + 2)
        if least is None or cost < least:
            best, least = kc, cost
    return best


# The chunk of the HEX8 operator is chosen at every launch of a solve, about ten
# times per iteration: tall meshes must not pay for a search over all their
# planes (0.4 ms and more for 60,000; a launch's own cost is a few microseconds).
@pytest.mark.parametrize("precision,resident", [(etm.ETM_PREC_FP64, 512), (etm.ETM_PREC_MIXED, 1024)])
def test_hex8_chunk_is_the_best_and_quick_to_choose(ask, precision, resident):
    shapes = [(1, 1, 1), (3, 3, 1), (30, 6, 2), (31, 7, 5), (97, 83, 33), (160, 152, 48), (256, 256, 64), (512, 512, 64),
              (1024, 1024, 128), (300, 300, 3), (32800, 7, 1), (8, 8, 499), (40, 36, 400), (31, 7, 6000), (7, 7, 20000),
              (1, 1, 60000)]
    for shape, (kc, ns) in zip(shapes, ask(["chunk %d %d %d %d" % (precision, *s) for s in shapes])):
        assert kc == hex8_chunk(*shape, resident), (shape, kc)
        assert ns < 100000, (shape, ns)
