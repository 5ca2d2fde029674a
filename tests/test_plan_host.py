"""Host logic of the plan (crf_plan.cpp), built for the CPU with stub HIP
allocation calls (tests/plan_host_stub.cpp) and checked on synthetic batches:
every sentence in exactly one inside and one CKY bundle, each bundle within
the launch's LDS, the chart layouts' stride congruences (the condition under
which the sweeps' LDS reads are bank-conflict free), the fused queue of the
no-allocation call, and the tile charts' bundles and workspace charts.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2008_03736_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM_INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir(ROCM_INCLUDE):
        pytest.skip("needs g++ and the HIP headers")
    out = str(tmp_path_factory.mktemp("plan") / "plan_host")
    # host code only (g++, no GPU code): built with the address and
    # undefined-behaviour sanitizers, which abort the run on a finding
    cmd = [cxx, "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM_INCLUDE,
           "-I" + os.path.join(HERE, "..", "include"), "-o", out, os.path.join(HERE, "plan_host_stub.cpp")]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    return out


def plan_of(harness, tmp_path, lengths, labels=None, flags=0):
    f = tmp_path / "lengths.txt"
    f.write_text("\n".join(str(int(v)) for v in lengths))
    args = [harness, str(f), str(labels if labels is not None else 1), str(flags)]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    res = subprocess.run(args, capture_output=True, text=True, env=env)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert "runtime error" not in res.stderr and "AddressSanitizer" not in res.stderr, res.stderr[-4000:]
    head, recs = None, []
    for line in res.stdout.splitlines():
        t = line.split()
        if t[0] == "P":
            head = dict(zip(["n_mix", "grid", "lds_in", "lds_ck", "half_cu"], map(int, t[1:])))
        elif t[0] == "W":
            head.update(zip(["spill", "cky_spill", "split_ws", "ws_users", "ws_bytes", "fused_queue"],
                            map(int, t[1:])))
        elif t[0] == "R":
            v = list(map(int, t[1:]))
            recs.append(dict(kind=v[0], n=v[1], count=v[2], split_ws=v[3], strict=v[4], ld=v[5], cs=v[6],
                             e=v[7], bytes=v[8], ids=v[9:]))
        elif t[0] == "I":
            v = list(map(int, t[1:]))
            recs.append(dict(kind=1, n=v[0], count=v[1], ids=v[2:]))
        elif t[0] == "Q":
            head.update(zip(["team_cap", "team_area"], map(int, t[1:])))
        elif t[0] == "T":
            v = list(map(int, t[1:]))
            head["n1"] = v[0]
            head.setdefault("tiles", []).append(v[1:])
        elif t[0] == "G":
            head.update(zip(["tile_on", "tile_long", "tile_scratch", "tile_cky", "tile_threads", "scratch_bytes",
                             "mbr_fused", "info_lds_in", "info_lds_ck"], map(int, t[1:])))
        elif t[0] == "B":
            v = list(map(int, t[1:]))
            head.setdefault("bundles", []).append(dict(launch=v[0], kind=v[1], m=v[2], count=v[3], pitch=v[4], lds=v[5],
                                                       used=v[6], pieces=v[7], ids=v[8::2], lens=v[9::2]))
        elif t[0] == "X":
            head.setdefault("ws_tiles", []).append(tuple(map(int, t[1:])))
        elif t[0] == "V":
            head.setdefault("ws_spans", []).append(tuple(map(int, t[1:])))
    return head, recs


def check_plan(head, recs, lengths):
    lengths = np.asarray(lengths)
    assert head["n_mix"] == len(recs)
    # one workgroup slot per CU per bundle LDS that fits (256 CUs, 160 KiB each)
    per_cu = min(4, max(1, 163840 // max(head["lds_in"], head["lds_ck"])))
    assert head["grid"] == min(len(recs), 256 * per_cu)
    for kind in (0, 1):
        ids = [i for r in recs if r["kind"] == kind for i in r["ids"]]
        assert sorted(ids) == list(range(len(lengths))), "every sentence once per kind"
    for r in recs:
        assert r["count"] == len(r["ids"]) >= 1
        assert all(lengths[i] == r["n"] for i in r["ids"])
        n, nb, ld, cs = r["n"], r["count"], r["ld"], r["cs"]
        if r["kind"] == 1:
            assert ld >= n + 1 and 2 * ld * ld <= cs < 2 * ld * ld + 32
            assert 0 < r["bytes"] <= head["lds_in"] <= 2 * head["half_cu"] + 256
            if r["strict"] and r["e"] == 0 and not (nb >= 32 and nb % 4 == 0):
                # span g's runs start at sigma g (mod 32): cs = sigma odd, ld = nb sigma
                assert cs % 2 == 1 and (ld - nb * cs) % 32 == 0, r
        else:
            assert ld >= n + 1 and cs % 8 == 0 and cs >= 8 * ld * ld
            u = cs // 8
            if r["strict"] and not (nb >= 16 and nb % 4 == 0):
                assert u % 2 == 1 and (ld + 1 - nb * u) % 16 == 0, r
            elif not r["strict"]:
                assert u % 2 == 1 and ld % 2 == 0


@pytest.mark.parametrize("name", ["tiny", "mixed", "longer"])
def test_plan_of_workloads(harness, tmp_path, name):
    b = W.make(name)
    head, recs = plan_of(harness, tmp_path, b.lengths)
    check_plan(head, recs, b.lengths)
    if name == "longer":
        # sentences of more than 99 words need a whole CU in either layout:
        # the launch runs one workgroup per CU, and those bundles take the
        # strict layout there
        assert head["lds_in"] > head["half_cu"]
        assert all(r["strict"] for r in recs if r["kind"] == 1 and r["n"] > 99)
    if name == "mixed":
        assert head["lds_in"] <= head["half_cu"]
        # both layouts occur, and most bundles take the strict one
        for kind in (0, 1):
            flags = [r["strict"] for r in recs if r["kind"] == kind]
            assert 0 < sum(flags) and sum(flags) > len(flags) // 2


@pytest.mark.parametrize("seed", range(6))
def test_plan_of_random_batches(harness, tmp_path, seed):
    rng = np.random.default_rng(seed)
    lengths = rng.integers(1, 100, size=int(rng.integers(1, 3000)))
    head, recs = plan_of(harness, tmp_path, lengths)
    check_plan(head, recs, lengths)


@pytest.mark.parametrize("n,count", [(9, 4), (14, 40), (17, 32), (20, 20), (30, 8), (45, 4), (99, 1)])
def test_plan_of_one_length(harness, tmp_path, n, count):
    lengths = [n] * count + [99] * 200
    head, recs = plan_of(harness, tmp_path, lengths)
    check_plan(head, recs, lengths)


@pytest.mark.parametrize("labels,seed", [(2, 0), (7, 1), (32, 2), (33, 3), (100, 4)])
def test_plan_of_labelled_batches(harness, tmp_path, labels, seed):
    # labelled plans run inside bundles only (no fused queue); each sentence
    # in exactly one bundle of sentences of its own length
    rng = np.random.default_rng(seed)
    lengths = rng.integers(1, 100, size=int(rng.integers(1, 2000)))
    head, recs = plan_of(harness, tmp_path, lengths, labels)
    assert head["n_mix"] == 0 and recs
    ids = [i for r in recs for i in r["ids"]]
    assert sorted(ids) == list(range(len(lengths)))
    for r in recs:
        assert r["count"] == len(r["ids"]) >= 1
        assert all(lengths[i] == r["n"] for i in r["ids"])


def test_workspace_users_reported(harness, tmp_path):
    # The mixed batch keeps every chart in LDS, yet its 99-word sentence's CKY
    # split table lives in the plan's workspace: plan info must count it as a
    # workspace user (calls on one plan are stream-ordered for that reason).
    b = W.make("mixed")
    head, _ = plan_of(harness, tmp_path, b.lengths)
    assert head["spill"] == 0 and head["cky_spill"] == 0
    long_ones = int(np.sum(b.lengths >= 97))
    assert long_ones >= 1
    assert head["split_ws"] == long_ones and head["ws_users"] == long_ones
    assert head["ws_bytes"] > 0
    # a batch of short sentences uses no workspace at all
    head, _ = plan_of(harness, tmp_path, [5, 9, 30, 60] * 10)
    assert head["ws_users"] == 0 and head["ws_bytes"] == 0
    # sentences past the LDS limit use it for both charts
    head, _ = plan_of(harness, tmp_path, [200, 150, 10])
    assert head["spill"] == 2 and head["cky_spill"] == 2 and head["ws_users"] == 2


def test_team_area_only_with_workspace_sentences(harness, tmp_path):
    # the team area (and the device's capacity for workspace workgroups: the
    # stub's 256 CUs, one workgroup each) exists exactly when some sentence's
    # chart is in the workspace
    head, _ = plan_of(harness, tmp_path, [200, 150, 10])
    assert head["team_area"] == 1 and head["team_cap"] == 256
    head, _ = plan_of(harness, tmp_path, W.make("mixed").lengths)
    assert head["team_area"] == 0
    # CRF_NO_TEAMS (0x2): workspace sentences, no team area
    head, _ = plan_of(harness, tmp_path, [200, 150, 10], flags=2)
    assert head["team_area"] == 0 and head["spill"] == 2


def test_step_shape_runs(harness):
    # shape_run_end, the closed form the sweeps use to run a shape's steps as
    # one loop, agrees with step_shape_k for every step up to 5000 splits:
    # the shape holds from K to the run's end and changes there
    res = subprocess.run([harness, "runs"], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "RUNS OK", res.stdout[-500:]


def test_tile_products_read_inside_the_charts(harness):
    # a lane that shares a tile and has no product left still loads: its
    # reads, like those of real products, stay inside the bundle's two squares
    res = subprocess.run([harness, "tilereads"], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.startswith("READS OK"), res.stdout[-500:]


def test_team_launch_shapes(harness):
    # Every workspace launch shape: a team of k (a power of two in
    # [kTeamMinK, kTeamMaxK] = [8, 16]) per job, m = ceil(jobs / 8) teams per
    # XCD, the grid 8 m k within what the device holds at once; otherwise a
    # workgroup per job.  Teams whenever the device has room for k >= 8.
    res = subprocess.run([harness, "teams"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    rows = [tuple(map(int, l.split()[1:])) for l in res.stdout.splitlines() if l.startswith("S ")]
    assert len(rows) == 8 * 301
    for jobs, cap, k, grid in rows:
        m = -(-jobs // 8)
        if k == 1:
            assert grid == jobs
            assert jobs == 0 or 8 * m * 8 > cap        # no room for teams of 8
        else:
            assert k in (8, 16) and grid == 8 * m * k <= cap
            assert 8 * m >= jobs and 8 * m <= 1024    # a team per job, within the team area
            assert k == 16 or 8 * m * 16 > cap        # the largest team that fits
    assert any(k > 1 for _, _, k, _ in rows)
    assert res.stdout.splitlines()[-1] == "N 1 5"     # no team area: a workgroup per job


SCRATCH_WS = (8 << 20) - 256   # the no-allocation call's workspace


def check_tile_charts(head, lengths, teams=False, force=False):
    """The tile charts' schedule: every sentence of up to 139 words in one
    bundle of each launch and kind, of its own block count, within the LDS of
    the launch (two workgroups a CU, or one), the lanes and the score pieces a
    thread keeps; the others on charts of their own in the workspace.  teams:
    sentences of more than 141 words are left to the kernels of single spans."""
    lengths = np.asarray(lengths)
    in_lds = np.flatnonzero(lengths <= 139) if not force else np.array([], int)
    on_spans = np.flatnonzero((lengths > 141) | force) if teams else np.array([], int)
    in_ws = np.setdiff1d(np.setdiff1d(np.arange(len(lengths)), in_lds), on_spans)
    assert head["tile_on"] == 1 and head["tile_long"] == (0 if teams else 1)
    bundles = head.get("bundles", [])
    for launch, kinds in ((0, [1]), (1, [0]), (2, [0, 1])):
        here = [r for r in bundles if r["launch"] == launch]
        for kind in kinds:
            assert sorted(i for r in here if r["kind"] == kind for i in r["ids"]) == list(in_lds)
        assert sorted({r["kind"] for r in here}) == (kinds if len(in_lds) else [])
    if len(in_lds) and len(in_ws):   # one launch holds both
        assert head["tile_threads"] == 512
    budget = head["half_cu"] if head["tile_threads"] == 256 else 163840 - 512
    for r in bundles:
        assert r["count"] == len(r["ids"]) >= 1 and [lengths[i] for i in r["ids"]] == r["lens"]
        assert all(n // 4 + 1 == r["m"] for n in r["lens"])
        assert r["used"] <= r["lds"] <= budget
        assert r["m"] * r["count"] <= head["tile_threads"] or r["count"] == 1
        if r["kind"] == 1:
            assert r["pieces"] <= 6 * head["tile_threads"]
            assert r["pitch"] >= r["m"] * r["count"] and (r["pitch"] % 2 == 0 or r["count"] == 1)
        if r["launch"] == 0:   # MBR decoding runs CKY in the inside bundle's LDS
            assert r["count"] * (72 * r["m"] * (r["m"] + 1) + 8) <= r["lds"]
    charts = head.get("ws_tiles", [])
    for kind in (0, 1):
        assert sorted(c[4] for c in charts if c[0] == kind) == list(in_ws)
    assert all(c[5] == lengths[c[4]] and c[1] == c[5] // 4 + 1 for c in charts)
    spans = [(c[2], c[3]) for c in charts]
    if teams:
        assert sorted(v[0] for v in head["ws_spans"]) == sorted(v[1] for v in head["ws_spans"]) == list(on_spans)
        spans.append((0, head["scratch_bytes"]))   # their charts, in use at the same time
    spans.sort()
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:])) and (not spans or spans[-1][1] <= head["ws_bytes"])
    assert head["spill"] == len(in_ws) + len(on_spans)
    # CKY alone: a width a step unless the sentences are short or some fit in
    # LDS neither way (teams take those a width a step too)
    assert head["tile_cky"] == int(lengths.max() <= 28 or (not teams and (force or lengths.max() > 141)))
    assert head["cky_spill"] == (head["spill"] if head["tile_cky"] else len(on_spans))
    if head["tile_cky"]:
        assert head["ws_users"] == head["spill"] and head["split_ws"] == 0
    else:
        assert head["ws_users"] == len(on_spans) + head["split_ws"]
        assert head["split_ws"] == np.sum(np.delete(lengths, on_spans) >= 96)
    assert head["mbr_fused"] == (1 if len(in_lds) else 0)
    # what does not fit the scratch as tiles runs on the fused queue, which must be there
    need = max([c[3] for c in charts], default=0)
    assert head["tile_scratch"] == (0 if need > SCRATCH_WS else 1)
    if not head["tile_scratch"] and head["scratch_bytes"] <= SCRATCH_WS:
        assert head["n_mix"] > 0 or len(in_lds) + np.sum(lengths[in_ws] <= 141) == 0


@pytest.mark.parametrize("name", ["tiny", "mixed", "longer", "stress"])
def test_tile_charts_of_workloads(harness, tmp_path, name):
    lengths = W.make(name).lengths
    head, _ = plan_of(harness, tmp_path, lengths)
    check_tile_charts(head, lengths)


@pytest.mark.parametrize("seed", range(8))
def test_tile_charts_of_random_batches(harness, tmp_path, seed):
    rng = np.random.default_rng(100 + seed)
    lengths = rng.integers(1, [8, 30, 99, 100, 139, 142, 200, 400][seed] + 1, size=int(rng.integers(1, 1500)))
    head, _ = plan_of(harness, tmp_path, lengths)
    check_tile_charts(head, lengths)


@pytest.mark.parametrize("lengths,flags,teams", [
    ([450] * 3 + [30], 0, False),              # up to 450 words: tiles
    ([451, 30], 0, True),
    ([460, 141, 150, 30], 0, True),            # 140 and 141 words: tile charts behind the others' charts
    ([500, 140, 141, 142, 143, 139, 5], 0, True),   # 142 words: not in both
    ([451] + [256] * 15, 0, True),             # 16 past LDS: teams
    ([451] + [256] * 16, 0, False),            # 17: tiles
    ([1023], 0, True),
    ([1023] * 20, 0, False),
    ([460, 141, 150, 30], 2, True),            # CRF_NO_TEAMS: the same kernels, a workgroup a pass, for the same bits
    ([460, 141, 150, 30], 1, True),            # CRF_FORCE_SPILL
    ([200, 141, 150, 30], 1, False),
])
def test_tile_charts_or_teams(harness, tmp_path, lengths, flags, teams):
    head, _ = plan_of(harness, tmp_path, lengths, flags=flags)
    check_tile_charts(head, lengths, teams, force=(flags & 1) != 0)


def test_tile_charts_past_the_scratch(harness, tmp_path):
    # sentences of 140 and 141 words keep their charts of single spans in LDS, so
    # that a plan can fit the no-allocation call's scratch on those alone
    lengths = [141] * 40 + [30] * 100
    head, _ = plan_of(harness, tmp_path, lengths)
    check_tile_charts(head, lengths)
    assert not head["tile_scratch"] and head["scratch_bytes"] <= SCRATCH_WS and head["n_mix"] > 0


def check_tiles(head, lengths, rows=64):
    """The scorer's tiles cover every valid cell (i < j <= n_b) of every
    sentence exactly once; a tile's rows and columns are fence posts of the
    batch (or -1); a tile that packs whole sentences uses its fence posts as
    both its rows and its columns."""
    lengths = np.asarray(lengths, np.int64)
    n1 = head["n1"]
    t = np.asarray(head["tiles"], np.int64)
    assert t.shape[1] == 2 * rows
    r, c = t[:, :rows], t[:, rows:]
    for ids in (r, c):
        v = ids[ids >= 0]
        assert np.all(v % n1 <= lengths[v // n1]), "a tile names a fence post past its sentence"
    rr = np.repeat(r[:, :, None], rows, axis=2)
    cc = np.repeat(c[:, None, :], rows, axis=1)
    ok = (rr >= 0) & (cc >= 0) & (rr // n1 == cc // n1) & (rr % n1 < cc % n1)
    cells = rr[ok] * n1 + cc[ok] % n1                       # (b n1 + i) n1 + j
    got = np.bincount(cells, minlength=len(lengths) * n1 * n1)
    b, i, j = np.unravel_index(np.arange(len(lengths) * n1 * n1), (len(lengths), n1, n1))
    want = ((i < j) & (j <= lengths[b])).astype(np.int64)
    assert np.array_equal(got, want), "valid cells covered exactly once, nothing else"
    # a sentence of up to rows - 1 words sits whole in one tile, whose rows
    # are also its columns
    short = np.flatnonzero(lengths + 1 <= rows)
    for k in range(len(t)):
        row = r[k][r[k] >= 0]
        for b in np.unique(row // n1):
            if lengths[b] + 1 <= rows:
                assert np.array_equal(np.sort(row[row // n1 == b] % n1), np.arange(lengths[b] + 1)), (k, b)
                assert np.array_equal(r[k], c[k])
    seen = np.unique(r[r >= 0] // n1)
    assert np.all(np.isin(short, seen))
    tile_idx = np.arange(len(t))[:, None].repeat(rows, 1)
    pairs = np.unique(np.stack([tile_idx[r >= 0], r[r >= 0] // n1], -1), axis=0)   # (tile, sentence)
    tiles_of = np.bincount(pairs[:, 1], minlength=len(lengths))
    assert np.all(tiles_of[short] == 1), "a short sentence in more than one tile"


@pytest.mark.parametrize("name", ["tiny", "mixed", "longer", "stress"])
def test_biaffine_tiles_cover_every_cell_once(harness, tmp_path, name):
    lengths = W.make(name, 0).lengths
    head, _ = plan_of(harness, tmp_path, lengths)
    check_tiles(head, lengths)


def test_biaffine_tiles_edge_lengths(harness, tmp_path):
    # one word, exactly a tile's rows (63 words: 64 fence posts), one past it,
    # two and three blocks, and many short sentences that fill tiles unevenly
    lengths = [1, 63, 64, 127, 128, 129, 200, 2, 3, 5, 7, 11, 13] + [4] * 40
    head, _ = plan_of(harness, tmp_path, lengths)
    check_tiles(head, lengths)
