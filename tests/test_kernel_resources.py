"""Register budgets of the HIP kernels, from the resource report that the
build writes beside the library (the compiler's per-kernel figures).

A kernel that runs out of registers spills to scratch memory: the spill
reloads then sit on the sweeps' dependent chain of steps and the spills add
HBM traffic (label code once compiled into the shared inside body pushed
every inside kernel past its 128 VGPRs and slowed the fused launch by a
fifth).  These tests hold every kernel to the scratch it uses now, so such a
change fails on the CPU, at build time, rather than in a profile."""
import csv
import os

import pytest

from paper_2008_03736_amd import build as BLD

# scratch bytes per lane each kernel may use; every other kernel none.  The
# fused kernel of the charts of single spans (both the inside and the CKY body
# in one persistent kernel) sits at 128 VGPRs with nothing spilled, since log Z
# is taken without a float64 log, whose coefficients a persistent loop would
# keep in registers (each spilled dword was stored once per lane, 1 MB of HBM
# writes per launch).  Only two team builds of the workspace kernels spill
# (their team state and job loop beside two full sweeps); they run on launches
# of a few long sentences, whose time is set by memory round trips.
ALLOWED_SCRATCH = {"spill_parse_kernel<true>": 72, "loss_kernel<true>": 20}
# every kernel the library launches (short names)
# (the workspace kernels come in a lone-workgroup and a team build: the
# last template argument)
EXPECTED = [
    "inside_kernel<false, false, true, false>", "inside_kernel<true, false, true, false>",
    "inside_kernel<false, true, false, false>", "inside_kernel<true, true, false, false>",
    "inside_kernel<false, true, false, true>", "inside_kernel<true, true, false, true>",
    "cky_kernel<false, false, false>", "cky_kernel<false, true, false>",
    "cky_kernel<true, false, false>", "cky_kernel<true, true, false>",
    "cky_kernel<true, false, true>", "cky_kernel<true, true, true>",
    "loss_kernel<false>", "loss_kernel<true>",
    "parse_kernel", "spill_parse_kernel<false>", "spill_parse_kernel<true>",
    "label_reduce_kernel", "label_expand_kernel", "label_spans_kernel", "zero_words",
    "tile_inside_kernel<false>", "tile_inside_kernel<true>", "tile_loss_kernel", "tile_cky_kernel",
    "tile_parse_kernel", "tile_mbr_kernel",
    "tile_ws_inside_kernel<false>", "tile_ws_inside_kernel<true>", "tile_ws_loss_kernel", "tile_ws_cky_kernel",
    "tile_ws_parse_kernel", "tile_ws_mbr_kernel",
    "tile_both_inside_kernel<false>", "tile_both_inside_kernel<true>", "tile_both_loss_kernel", "tile_both_cky_kernel",
    "tile_both_parse_kernel", "tile_both_mbr_kernel",
]


def short(name):
    name = name.replace("crf::(anonymous namespace)::", "").replace("crf::", "")
    if name.startswith("void "):
        name = name[5:]
    return name.split("(")[0]


@pytest.fixture(scope="module")
def report():
    if not os.path.exists(BLD.RESOURCES):
        pytest.fail("no kernel resource report: build the library (__graft_entry__.build())")
    with open(BLD.RESOURCES) as f:
        rows = list(csv.DictReader(f, delimiter="\t"))
    return {short(r["kernel"]): r for r in rows}


def test_report_lists_every_kernel(report):
    # every kernel that is launched, and no other
    scorers = {k for k in report if k.startswith(("biaffine_kernel<", "biaffine_small_kernel<"))}
    assert {k.split("<")[0] for k in scorers} == {"biaffine_kernel", "biaffine_small_kernel"}
    assert set(report) - scorers == set(EXPECTED)


def test_no_kernel_spills_beyond_its_budget(report):
    over = []
    for k, r in report.items():
        scratch = int(r["ScratchSize [bytes/lane]"])
        if scratch > ALLOWED_SCRATCH.get(k, 0):
            over.append(f"{k}: {scratch} bytes/lane of scratch ({r['VGPRs Spill']} VGPRs spilled)")
    assert not over, "kernels spill to scratch: " + "; ".join(over)


def test_kernels_keep_their_occupancy(report):
    # waves a SIMD: the charts of single spans five (forward only) and four,
    # the tile charts two (two workgroups of four wavefronts a CU, or one of
    # eight), those in the workspace at least the two of their one workgroup
    for k in report:
        least = 0
        if k == "inside_kernel<false, false, true, false>":
            least = 5
        elif k in ("inside_kernel<true, false, true, false>", "parse_kernel"):
            least = 4
        elif k.startswith("tile_"):
            least = 2
        assert int(report[k]["Occupancy [waves/SIMD]"]) >= least, k
