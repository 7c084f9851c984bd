"""The dispatch planners' choices and invariants, on the CPU.

tests/planner_probe.hip includes the library's dispatch source and prints
the split plan of the large-M kernel (plan_splits) and the few-row
streaming kernel's plan (stream_plan) for calls given as text.  Checked here:

* invariants every plan must keep for the kernels to be correct: parts of
  whole scale groups (4 steps of 64 k, or 8-block groups for the streaming
  kernel), no empty part, every step covered, at most 4 parts summed in the
  kernel and 16 by the separate launch, no split of a layer with a tile for
  every CU;
* the plans the design documents for its workloads: the q4 step block
  unsplit; single 128-tile layers at 2048 tokens in 2 parts (summed by the
  separate launch with an epilogue, in the kernel without); a d = 1024
  block at 768 tokens summed in the kernel with FFN-down in 4 parts; the
  paper widths at 214 tokens summed by the separate launch.

The probe is built with hipcc against the library's objects (built by
`python -m paper_2607_08526_amd.build`); without a GPU the planners assume
the 256 compute units of the target part.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

import kgroup_cases
import test_gpu_dit_chain
import test_gpu_epilogue
import test_gpu_parity
import test_zz_no_alloc

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
BUILD = os.path.join(ROOT, "paper_2607_08526_amd", "_build")
CUS = 256
INT8, Q4 = 8, 4


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not available")
    objs = [os.path.join(BUILD, f) for f in sorted(os.listdir(BUILD))
            if f.endswith(".o") and f != "qlinear.o"] if os.path.isdir(BUILD) else []
    if not objs:
        pytest.fail("library objects missing: run `python -m paper_2607_08526_amd.build`")
    out = tmp_path_factory.mktemp("probe")
    obj, exe = str(out / "probe.o"), str(out / "probe")
    flags = ["--offload-arch=gfx950", "-O1", "-std=c++17", f"-I{os.path.join(ROOT, 'include')}",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
    for cmd in ([hipcc, *flags, "-c", os.path.join(HERE, "planner_probe.hip"), "-o", obj],
                [hipcc, "--offload-arch=gfx950", "-o", exe, obj, *objs]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]

    def run(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return [l.split() for l in r.stdout.strip().splitlines()]
    return run


def wide_plans(probe, calls):
    """calls: (fmt, epi, M, [(N, K), ...]) -> [(ext, [(K, tiles, S, psteps), ...])]"""
    out = probe([f"wide {f} {int(e)} {M} " + " ".join(f"{N} {K}" for N, K in ls)
                 for f, e, M, ls in calls])
    res = []
    for t in out:
        assert t[0] == "wide"
        v = list(map(int, t[2:]))
        res.append((int(t[1]), [tuple(v[i:i + 4]) for i in range(0, len(v), 4)]))
    return res


def block(d):
    return [(3 * d, d), (d, d), (4 * d, d), (d, 4 * d)]


def test_wide_plans_keep_the_kernel_invariants(probe):
    rng = np.random.default_rng(0)
    calls = []
    for _ in range(300):
        M = int(rng.integers(65, 4097))
        fmt, epi = int(rng.choice([INT8, Q4])), bool(rng.integers(0, 2))
        if rng.random() < 0.5:
            d = 256 * int(rng.integers(1, 13))
            calls.append((fmt, epi, M, block(d)))
        else:
            n = int(rng.integers(1, 5))
            calls.append((fmt, epi, M, [(int(rng.integers(1, 65)) * 64,
                                         256 * int(rng.integers(1, 33))) for _ in range(n)]))
    for (fmt, epi, M, ls), (ext, layers) in zip(calls, wide_plans(probe, calls)):
        for K, tiles, S, ps in layers:
            ns = K // 64
            what = (fmt, epi, M, ls, ext, K, S, ps)
            assert S >= 1 and ps >= 1, what
            assert (S - 1) * ps < ns <= S * ps, what        # every step, no empty part
            if S > 1:
                assert ps % 4 == 0, what                     # whole scale groups
                assert S <= (16 if ext else 4), what         # sum launch / in-kernel bound
                assert tiles < CUS, what                     # a tile per CU: never split
        assert ext in (0, 1)


def test_wide_plans_of_the_documented_workloads(probe):
    step, single_epi, single_plain, qkv, mid, widths = wide_plans(probe, [
        (Q4, False, 2048, block(2048)),
        (Q4, True, 2048, [(2048, 8192)]),
        (Q4, False, 2048, [(2048, 2048)]),
        (Q4, True, 2048, [(6144, 2048)]),
        (Q4, True, 768, block(1024)),
        (Q4, False, 214, block(1024)),
    ])
    assert all(S == 1 for _, _, S, _ in step[1])           # the step block: unsplit
    assert single_epi == (1, [(8192, 128, 2, 64)])        # FFN-down alone, epilogue
    assert single_plain == (0, [(2048, 128, 2, 16)])      # out-projection alone, plain
    assert qkv[1][0][2] == 1                              # 384 tiles: whole
    assert mid[0] == 0 and [S for _, _, S, _ in mid[1]] == [4, 2, 2, 2]
    assert widths[0] == 1 and widths[1][0][:3] == (4096, 8, 8)


def test_stream_plans_keep_the_kernel_invariants(probe):
    rng = np.random.default_rng(1)
    calls = []
    for _ in range(200):
        M = int(rng.integers(1, 33))
        fmt = int(rng.choice([INT8, Q4]))
        n = int(rng.integers(1, 5))
        ls = [(int(rng.integers(1, 257)) * 32, 256 * int(rng.integers(1, 49))) for _ in range(n)]
        calls.append((fmt, M, ls))
    out = probe([f"stream {f} {M} " + " ".join(f"{N} {K}" for N, K in ls) for f, M, ls in calls])
    for (fmt, M, ls), t in zip(calls, out):
        assert t[0] == "stream"
        rw, kw, mx = map(int, t[1:4])
        assert rw in (8, 16, 32, 64) and kw in (2, 4, 8) and M <= mx <= 32, (t, M)
        v = list(map(int, t[4:]))
        for K, S, pb in (v[i:i + 3] for i in range(0, len(v), 3)):
            nb = K // 32
            what = (fmt, M, ls, t)
            assert 1 <= S <= 16, what
            assert pb % 8 == 0 and pb >= 8 * kw or S == 1, what
            assert (S - 1) * pb < nb <= S * pb or (S == 1 and pb >= nb), what


def test_stream_plans_of_the_documented_workloads(probe):
    # the grouped d = 2048 block (QKV, out, FFN-up, FFN-down) at few rows:
    # int8 at M = 8 must not take 8-row workgroups, which tie with wider
    # ones in round trips but re-read the activations twice as often (the
    # plan's byte floor separates them); q4 at M = 8 keeps its 32-row plan
    lay = [(6144, 2048), (2048, 2048), (8192, 2048), (2048, 8192)]
    out = probe([f"stream {f} {M} " + " ".join(f"{N} {K}" for N, K in lay)
                 for f, M in ((INT8, 8), (Q4, 8), (INT8, 32))])
    i8, q4, i8_32 = ([int(x) for x in t[1:4]] for t in out)
    assert i8[0] >= 16 and i8[2] == 8, out[0]
    assert q4[0] == 32 and q4[2] == 8, out[1]
    assert i8_32[0] == 32 and i8_32[2] == 32, out[2]


def kg_choices(probe, calls):
    """calls: (fmt, fp32 X, epilogue, M, [(N, K), ...]) -> [(use, [(K, shape,
    tile rows, tile columns), ...])]; use: the K-group kernel runs."""
    out = probe([f"kg {f} {int(x)} {int(e)} {M} " + " ".join(f"{N} {K}" for N, K in ls)
                 for f, x, e, M, ls in calls])
    res = []
    for t in out:
        assert t[0] == "kg"
        v = list(map(int, t[4:]))
        res.append((int(t[3]), [tuple(v[i:i + 4]) for i in range(0, len(v), 4)]))
    return res


def test_every_kgroup_shape_built_is_reached(probe):
    """Every shape that a launch of the K-group kernel holds is one that some
    call takes (single layers and groups of up to 8), and no call takes one it
    does not hold: bf16 X by the rows staged, fp32 X, fp16 weights."""
    rng = np.random.default_rng(4)
    calls = []
    for _ in range(4000):
        fmt, f32 = [(Q4, 0), (INT8, 0), (Q4, 1), (INT8, 1), (16, 0)][int(rng.integers(5))]
        M = int(round(np.exp(rng.uniform(0, np.log(600)))))
        n = int(rng.choice([1, 1, 2, 4, 8]))
        ls = [(int(np.exp(rng.uniform(3, 9.5))), 256 * int(np.exp(rng.uniform(0, 4))))
              for _ in range(n)]
        calls.append((fmt, f32, 0, M, ls))
    seen = {}
    for (fmt, f32, _, M, _), (use, layers) in zip(calls, kg_choices(probe, calls)):
        if use:
            rows = "f32" if f32 else "f16" if fmt == 16 else min(r for r in (8, 16, 32, 4096)
                                                                 if M <= r)
            for _, shape, tm, tn in layers:
                assert tm > 0 and tn > 0, (fmt, f32, M)
                seen.setdefault((fmt, rows), set()).add(shape)
    for fmt in (Q4, INT8):
        for rows in (8, 16, 32):
            assert seen[fmt, rows] == ({0, 1, 2} if fmt == Q4 and rows < 32 else {0, 1, 2, 5})
        assert seen[fmt, 4096] == set(range(6))
        assert seen[fmt, "f32"] == {0, 1, 2, 3}
    assert seen[16, "f16"] == {0, 1, 2, 3}


def test_plans_are_made_once(probe):
    """A program's shapes (a model's layers and blocks at 40 clip lengths) are
    looked up, not planned again, and where the choice needed the large-M plan
    the launch finds that one too."""
    calls = [f"kg {Q4} 0 {e} {M} " + " ".join(f"{N} {K}" for N, K in ls)
             for M in range(70, 2030, 50) for e, ls in
             [(0, block(1024))] + [(1, [l]) for l in block(1536)]]
    out = probe(calls + calls)
    first, second = out[:len(calls)], out[len(calls):]
    assert all(t[1] == "0" for t in first)
    assert all(t[2] == "1" for t in first)
    assert all(t[1] == "1" for t in second)


def routes(probe, calls):
    """calls: (fmt, fp32 X, epilogue, forced path, [(M, N, K), ...]) ->
    [(kernel, [(K, shape or K parts), ...] in launch order)]"""
    out = probe([f"route {f} {int(x)} {int(e)} {p} " + " ".join(f"{M} {N} {K}" for M, N, K in ls)
                 for f, x, e, p, ls in calls])
    res = []
    for t in out:
        assert t[0] == "route"
        v = list(map(int, t[2:]))
        res.append((t[1], list(zip(v[::2], v[1::2]))))
    return res


AUTO, GEMV, STREAM, SKINNY, TILED, WIDE, MID = range(7)  # forced paths
F16 = 16


def test_forced_paths_reach_their_kernels(probe):
    """Each forced path, by format and activation type; fp16 weights follow the
    large-M path's value at any M and no other."""
    one = lambda M=8, N=300, K=1024: [(M, N, K)]
    for fmt in (Q4, INT8):
        want = [(GEMV, one(4), "rows", 0), (STREAM, one(), "rows", 1), (SKINNY, one(), "rows", 2),
                (TILED, one(), "tiled", None), (WIDE, one(), "wideext", None),
                (MID, one(), "mid", None), (MID, one(8, 300, 96), "refused", None),
                (WIDE, one(8, 300, 96), "refused", None)]
        got = routes(probe, [(fmt, 0, 0, p, ls) for p, ls, _, _ in want])
        for (p, ls, kernel, v), (k, vs) in zip(want, got):
            assert k == kernel and (v is None or vs[0][1] == v), (fmt, p, ls, k, vs)
        got = routes(probe, [(fmt, 1, 0, p, one()) for p in range(1, 7)])
        assert [k for k, _ in got] == ["refused"] * 3 + ["tiled"] + ["refused"] * 2
    for M in (1, 65, 300):
        auto = routes(probe, [(F16, 0, 0, AUTO, one(M))])
        got = routes(probe, [(F16, 0, 0, p, one(M)) for p in range(1, 7)])
        assert [g for g in got[:4] + got[5:]] == auto * 5
        assert got[4][0] in ("wide", "wideext")


def test_kgroup_cases_run_the_kgroup_kernel(probe):
    """The calls that test_gpu_kgroup.py makes, and the shapes they take."""
    groups = [((f, x, 0, AUTO, [(M, N, K) for N, K in ls]), sh)
              for f, x, M, ls, sh in kgroup_cases.GROUPS]
    for (c, sh), (kernel, v) in zip(groups, routes(probe, [c for c, _ in groups])):
        assert kernel == "kg" and [s for _, s in v] == sh, (c, kernel, v)
    singles = [(f, 0, 0, AUTO, [c]) for f in (Q4, INT8) for c in kgroup_cases.SINGLES]
    singles += [(f, x, 0, AUTO, [c]) for f, x in ((Q4, 1), (INT8, 1), (F16, 0))
                for c in kgroup_cases.SINGLES_F32_F16]
    singles += [(f, 1, 0, AUTO, [(64, 1024, 1024)]) for f in (Q4, INT8)]  # large activations
    singles += [(Q4, 0, 1, AUTO, [(M, N, K) for N, K in block(512)]) for M in (7, 30, 107)]
    for c, (kernel, v) in zip(singles, routes(probe, singles)):
        assert kernel == "kg", (c, kernel)


def test_gpu_tests_reach_what_they_are_for(probe):
    """The kernels, K parts and sum launches of GPU tests that are about them."""
    par, ep = test_gpu_parity, test_gpu_epilogue
    for fmt in (Q4, INT8):
        one = lambda path, M, N, K, epi=0: (fmt, 0, epi, path, [(M, N, K)])
        M, ls = par.SPLIT_GROUP
        want = [(one(WIDE, M_, *par.IN_KERNEL_NK), "wide", [4]) for M_ in par.IN_KERNEL_M]
        want += [(one(WIDE, *c), "wideext", None) for c in par.SPLIT_CASES]
        want += [((fmt, 0, 0, WIDE, [(M, N, K) for N, K in ls]), "wideext", [16, 2, 2])]
        want += [(one(p, *c), "mid" if p == MID else "wideext", None)
                 for c, p in par.REPLAY_CASES.values()]
        want += [(one(MID, *c), "mid", None) for c in par.MID_CASES]
        want += [(one(WIDE, *c), "wideext", None) for c in par.WORKSPACE_CASES]
        want += [((fmt, 0, 1, WIDE, [(384, N, K) for N, K in ep.ROUTED_GROUP]), "wideext",
                  [16, 16, 2, 2]),
                 ((fmt, 0, 1, AUTO, [(768, N, K) for N, K in block(1024)]), "wide", [4, 2, 2, 2]),
                 ((fmt, 0, 0, AUTO, par.MIXED_ROWS), "rows", [0, 0, 0, 1, 1, 0])]
        for M in (1, 3):
            want.append(((fmt, 0, 0, AUTO, [(M, N, K) for N, K in block(2048)]), "rows", [0] * 4))
        for M in (8, 32):
            want.append(((fmt, 0, 0, AUTO, [(M, N, K) for N, K in block(2048)]), "kg", None))
        for (c, kernel, v), (k, got) in zip(want, routes(probe, [c for c, _, _ in want])):
            assert k == kernel, (c, k)
            assert v is None or [x for _, x in got] == v, (c, got)
            if k in ("mid", "wideext") and c[4] != [(65, 130, 256)] and v is None:
                assert all(x > 1 or K < 1024 for K, x in got), (c, got)  # parts, in a workspace
    # the chained step's linears, one call each, and the steered block
    for (B, T, p), kernel in zip(test_gpu_dit_chain.CHAINS, ("wide", "kg", "rows")):
        got = routes(probe, [(Q4, 0, 1, p, [(B * T, N, K)]) for N, K in block(256)])
        assert all(k.startswith(kernel) for k, _ in got), (B, T, p, got)
    got = routes(probe, [(Q4, 0, 1, p, [(256, N, K) for N, K in block(512)]) for p in (AUTO, WIDE)])
    assert [k for k, _ in got] == ["kg", "wideext"], got
    names = {ep.GEMV: ("rows", 0), ep.STREAM: ("rows", 1), ep.SKINNY: ("rows", 2),
             ep.TILED: ("tiled", None), ep.WIDE: ("wide", None), ep.MID: ("mid", None),
             ep.AUTO: ("kg", None)}
    calls = [(f, x == 0, 1, p, [(M, N, K)]) for f, x, M, N, K, p in ep.PATHS]
    for c, (k, v) in zip(calls, routes(probe, calls)):
        kernel, which = names[c[3]]
        assert k.startswith(kernel) and (which is None or v[0][1] == which), (c, k, v)
    calls = [(Q4, 0, 1, p, [(M, N, K) for N, K in ls]) for M, ls, p in ep.EP_GROUPS]
    assert [k for k, _ in routes(probe, calls)] == ["wideext", "kg", "rows", "kg"]
    # the static scratch is used: pre-pass copies and partials, then partials
    (f0, d0, M0, p0), (f1, d1, M1, p1) = test_zz_no_alloc.TWO_CALLS
    got = routes(probe, [(f0, 0, 1, p0, [(M0, N, K) for N, K in block(d0)]),
                         (f1, 0, 1, p1, [(M1, N, K) for N, K in block(d1)])])
    assert [k for k, _ in got] == ["wideext", "rows"] and max(v for _, v in got[0][1]) > 1
    t = probe([f"stream {f1} {M1} " + " ".join(f"{N} {K}" for N, K in block(d1))])[0]
    assert max(map(int, t[5::3])) > 1, t


def test_one_stage_layers_at_few_rows(probe):
    """K = 256 at few rows: the streaming kernel's whole-layer plan (about 4.2
    us) is ahead of the K-group kernel (about 5), except where the columns fill
    the GPU several times over."""
    calls = [(f, 0, 0, M, ls) for f in (Q4, INT8) for M in (5, 8, 16, 32)
             for ls in ([(893, 256)], [(64, 256)], [(3000, 256)], block(256))]
    for c, (use, _) in zip(calls, kg_choices(probe, calls)):
        assert not use, c
    wide_n = [(INT8, 0, 0, 32, [(8775, 256)]), (Q4, 0, 0, 7, [(7552, 256)] * 3)]
    assert all(use for use, _ in kg_choices(probe, wide_n))


def test_q4_up_to_sixteen_rows(probe):
    """q4 at up to 16 rows: reductions of 1280 to 1536 stay streamed (5.4 to
    5.7 us against 5.9 to 6.4); shorter ones and the blocks take the K-group
    kernel."""
    calls = [(Q4, 0, 0, M, ls) for M in (9, 13, 16)
             for ls in ([(1025, 1280)], [(1574, 1536)], [(129, 1280)] * 3)]
    assert not any(use for use, _ in kg_choices(probe, calls))
    calls = [(Q4, 0, 0, M, ls) for M in (9, 16) for ls in (block(512), block(2048), [(300, 768)])]
    assert all(use for use, _ in kg_choices(probe, calls))


def test_int8_four_rows(probe):
    """int8 at four rows: the alternative is the GEMV, ahead on small launches
    (a d = 512 block 6.6 us against 7.5, one-stage layers 4.0 against 5.0); the
    larger blocks take the K-group kernel."""
    stay = [block(512), block(256), [(893, 256)], [(64, 256)], [(5605, 1280)], [(2048, 8192)]]
    take = [block(768), block(1024), block(1536), block(2048), [(4500, 256)], [(8198, 4096)]]
    calls = [(INT8, 0, 0, 4, ls) for ls in stay + take]
    got = [use for use, _ in kg_choices(probe, calls)]
    assert got == [0] * len(stay) + [1] * len(take), got


def test_fp32_activations(probe):
    """fp32 activations: few rows and a reduction of a few thousand, or many
    rows of one stage, stay with the tiled kernel (2816 to 4352 long at one to
    eight rows 9.5 to 12 us against 11 to 15); wider or shorter layers and the
    blocks take the K-group kernel."""
    stay = [(1, [(91, 4352)]), (8, [(754, 4096)]), (3, [(199, 3840)]), (15, [(97, 4352)]),
            (29, [(497, 4352)]), (8, [(2048, 8192)]), (518, [(2213, 256)] * 2),
            (416, [(5855, 256)]), (976, [(705, 256)] * 3)]
    take = [(64, [(1024, 1024)]), (16, [(4608, 1536)]), (1, [(63, 768)]), (8, block(1024)),
            (32, block(2048)), (30, block(256)), (200, [(2048, 2048)])]
    for fmt in (Q4, INT8):
        calls = [(fmt, 1, 0, M, ls) for M, ls in stay + take]
        got = [use for use, _ in kg_choices(probe, calls)]
        assert got == [0] * len(stay) + [1] * len(take), (fmt, got)


def test_w8a8_launches_fit_a_grid(probe):
    """A launch holds fewer than 2^32 threads: a product whose pipelined shapes
    all pass that keeps the general kernel, and any other one stays on the
    fastest shape that fits.  Scales at an odd 2-byte address, K that is not
    whole 64-k steps, and the single-step products that the general kernel is
    ahead on, take the general kernel."""
    GENERAL, LARGE, MID, SMALL = range(4)
    cases = [((0, 8, 1191, 64), GENERAL), ((0, 1, 168, 64), GENERAL), ((0, 9, 1191, 64), SMALL),
             ((0, 8, 1191, 128), SMALL), ((0, 1410, 3915, 64), GENERAL),
             ((0, 1410, 3916, 64), LARGE), ((0, 1759, 1097, 64), LARGE),
             ((0, 2 ** 30, 1, 64), GENERAL), ((0, 2 ** 30, 64, 64), GENERAL),
             ((0, 2 ** 30 - 128, 1, 64), LARGE), ((0, 2 ** 27, 128, 4096), LARGE),
             ((0, 2048, 8192, 2048), LARGE), ((0, 1290, 1536, 1536), MID),
             ((0, 64, 4608, 1536), SMALL), ((2, 1290, 1536, 1536), GENERAL),
             ((0, 1290, 1536, 1504), GENERAL)]
    out = probe(["w8a8 " + " ".join(map(str, c)) for c, _ in cases])
    for (c, kernel), t in zip(cases, out):
        k, wgs, threads = map(int, t[1:])
        assert k == kernel, (c, t)
        assert wgs * threads < 2 ** 32, (c, t)
