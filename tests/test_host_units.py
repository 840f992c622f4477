"""Host-side units built with the host compiler (no GPU, no HIP).

1. The C ABI's validation layer (validate.cpp, api.cpp) under the address
   and undefined-behaviour sanitizers, with stub kernel launches: every
   status code of include/starkv.h comes back where the header says.
2. The spatial-cell arithmetic of the statistics kernel (grid_cell.h, the
   same source the kernel compiles) against exact integer arithmetic, up to
   the largest frames the boundary accepts (rows * cols <= 2^26).
3. The statistics kernel's block-shape choice (stats_shape.h) on the
   workloads' shapes and around every threshold.
"""

import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_01790_amd", "csrc")
INC = os.path.join(ROOT, "include")
HOST = os.path.join(ROOT, "tests", "host")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


def _build(tmp_path, name, sources, sanitize):
    exe = str(tmp_path / name)
    cmd = ["g++", "-std=c++17", "-g", "-O1", f"-I{INC}", f"-I{CSRC}", *sources, "-o", exe]
    if sanitize:
        cmd[1:1] = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-fno-omit-frame-pointer"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def test_abi_validation_under_sanitizers(tmp_path):
    exe = _build(tmp_path, "abi_driver",
                 [os.path.join(HOST, "abi_driver.cpp"), os.path.join(CSRC, "validate.cpp"),
                  os.path.join(CSRC, "api.cpp")], sanitize=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "checks passed" in r.stdout
    codes = {int(line.rsplit("-> ", 1)[1]) for line in r.stdout.splitlines()
             if line.startswith("ok ") and "status string" not in line
             and "launch count" not in line and "bytes" not in line
             and "count" not in line}
    # every starkv_status value 0..10 occurs
    assert set(range(11)) <= codes, sorted(codes)


def _cells(exe, cases):
    inp = "".join(f"{p} {rows} {cols} {M}\n" for p, rows, cols, M in cases)
    r = subprocess.run([exe], input=inp, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]


def test_grid_cells_exact_at_large_positions(tmp_path):
    exe = _build(tmp_path, "grid_cell_driver", [os.path.join(HOST, "grid_cell_driver.cpp")],
                 sanitize=True)
    rnd = random.Random(5)
    cases = []
    big = 1 << 26                                   # largest span the boundary accepts
    small = 1 << 22                                 # the reciprocal-estimate path's limit
    for rows, cols in [(big, 1), (big // 2, 2), (big // 3, 3), (1, big), (8191, 8192),
                       (4096 * 4, 4096), (39, 69), (51, 91), (26, 46), (4000, 4000),
                       (3, big // 3), (7, 3), (1, 1), (1025, 1023), (2, 1024)]:
        n = rows * cols
        for M in (1, 7, 8, 16):
            pts = {0, n - 1, n // 2, n // 3, min(n - 1, 33554434), min(n - 1, (1 << 25) - 1),
                   min(n - 1, small - 1), min(n - 1, small), min(n - 1, 1023)}
            pts |= {rnd.randrange(n) for _ in range(40)}
            pts |= {rnd.randrange(min(n, 1024)) for _ in range(20)}
            cases += [(p, rows, cols, M) for p in sorted(pts)]
    got = _cells(exe, cases)
    assert len(got) == len(cases)
    for (p, rows, cols, M), (r, c, cell, ok) in zip(cases, got):
        assert (r, c) == divmod(p, cols), (p, rows, cols)
        want = (r * M // rows) * M + (c * M // cols)
        assert cell == want, (p, rows, cols, M, cell, want)
        assert 0 <= cell < M * M
        # the kernel's span-entry path: reciprocal estimates one ulp off
        assert ok == 1, (p, rows, cols, M)


def test_small_quotient_exact_near_every_multiple(tmp_path):
    exe = _build(tmp_path, "grid_cell_driver", [os.path.join(HOST, "grid_cell_driver.cpp")],
                 sanitize=False)
    r = subprocess.run([exe, "quot"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    bad, checked = map(int, r.stdout.split())
    assert checked > 10**6 and bad == 0, (bad, checked)


def test_statistics_block_shape(tmp_path):
    """Wide (1024) when every block fits one per CU or the bins need it;
    small (256) when even two per CU leave a second round and K <= 9,
    M*M <= 64; narrow (512) otherwise."""
    exe = _build(tmp_path, "stats_shape", [os.path.join(HOST, "stats_shape_driver.cpp")],
                 sanitize=False)
    cases = [
        # (blocks, CUs, K, M) -> shape
        ((28 * 6, 256, 8, 8), 1024),      # 28 layers, 4 groups: the five-frame trajectory
        ((28 * 33, 256, 8, 8), 256),      # per-head subspaces
        ((28 * 33, 256, 12, 8), 512),     # per-head, more bins than the small shape holds
        ((28 * 33, 256, 8, 9), 512),      # per-head, more cells than the small shape holds
        ((28 * 33, 256, 18, 8), 1024),    # more bins than the narrow shape holds
        ((48 * 6, 256, 8, 8), 512),       # between one and two blocks per CU
        ((96 * 6, 256, 9, 8), 256),
        ((96 * 6, 256, 10, 8), 512),
        ((96 * 6, 256, 8, 16), 512),
        ((256, 256, 17, 16), 1024),       # exactly one per CU
        ((257, 256, 17, 16), 512),
        ((512, 256, 9, 8), 512),          # exactly two per CU
        ((513, 256, 9, 8), 256),
        ((513, 256, 1, 1), 256),
        ((1, 1, 64, 16), 1024),
    ]
    inp = "".join(f"{b} {c} {k} {m}\n" for (b, c, k, m), _ in cases)
    r = subprocess.run([exe], input=inp, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = [int(x) for x in r.stdout.split()]
    assert got == [want for _, want in cases], list(zip(cases, got))
    # blocks per layer: one per subspace (MI), one AEB block, and one
    # stability block per eight subspaces (four groups: 6; 28 heads: 33)
    subs = [1, 4, 7, 8, 9, 16, 17, 28, 63, 64]
    r = subprocess.run([exe, "layer"], input="".join(f"{n}\n" for n in subs),
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    assert got == [(-(-n // 8), n + 1 - (-n // 8)) for n in subs], list(zip(subs, got))
    assert got[1][1] == 6 and got[7][1] == 33


def test_entropy_blocks(tmp_path):
    """Four entropy blocks per layer only where they were timed to be faster:
    long contexts, and launches of at most five blocks per four CUs."""
    exe = _build(tmp_path, "stats_shape", [os.path.join(HOST, "stats_shape_driver.cpp")],
                 sanitize=False)
    cases = [   # (Lp, entropy, layers, subspaces, CUs) -> blocks
        ((140254, 1, 1, 4, 256), 4), ((140254, 1, 28, 4, 256), 4),
        ((140254, 1, 35, 4, 256), 4),      # 315 blocks
        ((140254, 1, 36, 4, 256), 1),      # 324
        ((140254, 1, 23, 8, 256), 4), ((140254, 1, 25, 8, 256), 1),
        ((140254, 0, 28, 4, 256), 1),      # the confidence statistic
        ((98304, 1, 28, 4, 256), 4), ((98303, 1, 28, 4, 256), 1),
        ((35495, 1, 28, 4, 256), 1), ((35495, 1, 25, 8, 256), 1), ((1, 1, 1, 1, 1), 1),
    ]
    r = subprocess.run([exe, "entropy"], capture_output=True, text=True, timeout=60,
                       input="".join(" ".join(map(str, c)) + "\n" for c, _ in cases))
    assert r.returncode == 0, r.stderr
    got = [int(x) for x in r.stdout.split()]
    assert got == [want for _, want in cases], list(zip(cases, got))


def test_scoring_slab_division(tmp_path):
    """Every slab of every (layer, group) belongs to exactly one block of each
    pass, a group's records of pass 1 are numbered from 0 in block order and
    fit the workspace, and waves share a slab only where the block's slabs
    fit; over token counts around the slab and record sizes, group counts
    around the CU count, and all three divisions of each pass."""
    exe = _build(tmp_path, "slab_grid", [os.path.join(HOST, "slab_grid_driver.cpp")],
                 sanitize=True)
    lines = []
    for Lp in [1, 63, 64, 65, 255, 256, 257, 511, 2915, 13679, 40845, 140190]:
        for nlg in [1, 2, 3, 4, 7, 12, 64, 112, 255, 256, 257, 448, 1000]:
            for nrb in (1, 7, 8, 9, 14, 16):
                for n_cu in (256, 304, 1):
                    one = (Lp + nlg + nrb) % 2
                    lines.append((Lp, nlg, nrb, n_cu, -(-Lp // 256), one, 1 if one else nrb % 2))
    r = subprocess.run([exe], input="".join(" ".join(map(str, x)) + "\n" for x in lines),
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = r.stdout.splitlines()
    assert len(out) == len(lines)
    bad = [(x, o) for x, o in zip(lines, out) if not o.startswith("ok ")]
    assert not bad, bad[:10]
    for p in (1, 2):
        assert {o.split()[p] for o in out} == {"small", "aligned", "crossing"}


def _launches(tmp_path, lines, full=False):
    exe = _build(tmp_path, "slab_grid", [os.path.join(HOST, "slab_grid_driver.cpp")],
                 sanitize=False)
    r = subprocess.run([exe], input="".join(" ".join(map(str, x)) + "\n" for x in lines),
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    out = [line.split() for line in r.stdout.splitlines()]
    assert all(o[0] == "ok" for o in out) and len(out) == len(lines)
    return [(o[1], o[2], *map(int, o[3:6 if full else 5])) for o in out]


def test_scoring_division_between_frame_counts(tmp_path):
    """The division of each pass on 256 CUs where both were timed, one to
    twelve 1920x1080 frames (2,691 visual tokens each, 224 text tokens) on 4
    groups: aligned blocks where they were the faster, ranges crossing groups
    where those were, either where they are within 2% of each other."""
    frames = [1, 2, 3, 4, 5, 6, 7, 8, 10, 12]
    tok = [f * 2691 + 224 for f in frames]
    got = _launches(tmp_path, [(t, 28 * 4, 7, 256, -(-t // 256), 1, 1, 128, 2) for t in tok])
    pass1 = "aligned aligned aligned aligned aligned - - - crossing crossing".split()
    pass2 = "aligned aligned - crossing crossing crossing crossing crossing crossing crossing".split()
    for f, a, b, g in zip(frames, pass1, pass2, got):
        assert a in ("-", g[0]), (f, "pass 1", g)
        assert b in ("-", g[1]), (f, "pass 2", g)
    # three and five frames on 14 layers: pass 1 in one round of 4 blocks per
    # group, whose reference slab is no part of the rounds, not two rounds of 9
    got = _launches(tmp_path, [(t, 14 * 4, 7, 256, -(-t // 256), 1, 1, 128, 2) for t in (8297, 13679)])
    assert [g[2] for g in got] == [224, 224], got


def test_unrolled_pass_shares_no_slab(tmp_path):
    """The unrolled pass-2 kernel gives each wave whole slabs, so its division
    is estimated without waves sharing one; the rolled kernel's may share."""
    lines = [(Lp, nlg, nrb, n_cu, -(-Lp // 256), 1, 1, 128, 2)
             for Lp in (64, 700, 2915, 5606, 13679) for nlg in (2, 8, 16, 56, 112)
             for nrb in (1, 4, 7, 8) for n_cu in (256, 304)]
    _launches(tmp_path, lines)


def _form_launches(tmp_path, forms):
    """The launches on 256 CUs of (layers, H, G, d, W, Lp, dtype, per_head)
    scoring calls."""
    lines = []
    for nl, H, G, d, W, Lp, dtype, per_head in forms:
        one = not per_head or H == G
        lines.append((Lp, nl * G, -(-W * (H // G) // 32), 256, -(-Lp // 256), int(one),
                      int(one or W % 32 == 0), d, 4 if dtype == "f32" else 2))
    return [(*g[:2], g[4]) for g in _launches(tmp_path, lines, full=True)]


def test_score_forms_cross_groups(tmp_path):
    """The shapes that the GPU tests of crossing blocks use give crossing
    blocks in both passes."""
    from tests.test_score_paths_gpu import CROSSING
    assert set(_form_launches(tmp_path, CROSSING)) == {("crossing", "crossing", 1)}


def test_scoring_launch_rules(tmp_path):
    """Which launches take the small-call kernels and where waves share a
    slab, on both sides of every line drawn by timing, on 256 CUs."""
    form = lambda Lp, nlg, nrb, d, esz, one=1: (Lp, nlg, nrb, 256, -(-Lp // 256), one, 1, d, esz)
    cases = [   # (case, pass 1, pass 2, waves per slab of pass 2)
        (form(2915, 4, 7, 128, 2), "small", "small", None),       # 48 chunks, 184 slabs
        (form(2915, 8, 7, 128, 2), "small", "aligned", 1),        # 368 slabs
        (form(2915, 8, 7, 128, 2, 0), "small", "small", None),
        (form(2915, 8, 4, 128, 2, 0), "small", "aligned", 1),
        (form(2915, 8, 7, 64, 2), "small", "small", None),
        (form(2915, 12, 7, 64, 2), "small", "aligned", 1),
        (form(2915, 8, 1, 64, 2), "small", "aligned", 1),
        (form(700, 4, 2, 128, 2), "small", "aligned", 1),
        (form(700, 4, 3, 128, 2), "small", "small", None),
        (form(256 * 64, 4, 7, 128, 2), "small", "aligned", 1),    # 256 chunks
        (form(256 * 64 + 1, 4, 7, 128, 2), "aligned", "aligned", 1),
        (form(2915, 4, 14, 128, 2), "small", "small", None),
        (form(2915, 8, 14, 128, 2), "small", "aligned", 4),       # two slabs per block
        (form(2915, 12, 14, 128, 2), "small", "aligned", 1),      # three
        (form(2915, 4, 9, 128, 2), "aligned", "small", None),
        (form(2915, 8, 9, 128, 2), "aligned", "aligned", 1),
        (form(2915, 8, 9, 64, 2), "small", "aligned", 1),
        (form(2915, 8, 4, 64, 4), "small", "small", None),
        (form(2915, 8, 2, 64, 4), "small", "aligned", 2),
        (form(2915, 12, 2, 64, 4), "small", "aligned", 1),
    ]
    got = _launches(tmp_path, [c for c, *_ in cases], full=True)
    for (c, a, b, rs), g in zip(cases, got):
        assert (g[0], g[1]) == (a, b) and rs in (None, g[4]), (c, g)


def _aligned_blocks(S, nlg, n_cu, p_max, first, start):
    """Blocks per group of the cheapest aligned division, every count tried."""
    best = None
    for p in range(1, p_max + 1):
        q = -(-S // p)
        rounds = -(-p * nlg // n_cu)
        cost = rounds * (-(-(q - first) // 8) * 8 + start)
        if best is None or (cost, rounds, -p) < best[0]:
            best = ((cost, rounds, -p), p)
    return best[1]


def test_scoring_division_tries_the_counts_that_matter(tmp_path):
    """The division looks at four block counts per group, the largest of each
    number of rounds; the cheapest of all counts is among them."""
    lines, want = [], []
    for Lp in (1025, 2915, 5606, 8297, 13679, 40845):
        for nlg in (20, 40, 56, 90, 112, 200, 256, 300, 600, 1200):
            S, mc = -(-Lp // 64), -(-Lp // 256)
            lim = max(1, 4 * 256 // nlg)
            lines.append((Lp, nlg, 7, 256, mc, 1, 1, 128, 2))
            want.append((_aligned_blocks(S, nlg, 256, min(mc, S, lim), 1, 10),
                         _aligned_blocks(S, nlg, 256, min(S, lim), 0, 8)))
    seen = 0
    for x, w, g in zip(lines, want, _launches(tmp_path, lines, full=True)):
        for i in (0, 1):
            if g[i] == "aligned":
                assert g[2 + i] == w[i] * x[1], (x, i, w, g)
                seen += 1
    assert seen > 60, seen


def test_score_row_blocks_take_their_kernels(tmp_path):
    """The GPU tests of every row-block count and of shared slabs launch the
    kernels they name: the persistent ones, or the small-call ones."""
    from tests.test_score_paths_gpu import ROW_BLOCKS, SHARED, SMALL_ROW_BLOCKS
    for a, b, _ in _form_launches(tmp_path, ROW_BLOCKS):
        assert "small" not in (a, b)
    small = _form_launches(tmp_path, SMALL_ROW_BLOCKS)
    assert {f[1] for f in small} == {"small"} and {f[0] for f in small} == {"small", "aligned"}
    assert [f[1:] for f in _form_launches(tmp_path, SHARED)] == [("aligned", 4), ("aligned", 2)]
