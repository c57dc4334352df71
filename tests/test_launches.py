"""CPU: the kernels that calls launch and the order in which they do, through a
stand-in HIP runtime that records launches (launch_recorder.py)."""
import pytest

import launch_recorder


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return launch_recorder.start(tmp_path_factory.mktemp("recorder"))


@pytest.mark.parametrize("op", ["combine", "noalloc"])
def test_threads_sharing_a_workspace_do_not_split_a_call(recorder, op):
    """Host threads that enqueue calls on one stream with one workspace (the
    calls then never overlap in time): nothing another thread enqueues comes
    between the launches of a call, which hand the inverse map and Y over
    through the workspace, nor between the clear for a new layout and them."""
    got = launch_recorder.run(recorder, f'''
import threading
recorder.recorder_pause_us(300)
shapes = [dict(T=64, H=512, I=64, E=8, topk=2), dict(T=40, H=512, I=64, E=8, topk=2, C=3),
          dict(T=90, H=256, I=64, E=4, topk=2, mode=1)]
def work(i):
    for n in range(6):
        assert call("{op}", **shapes[(i + n) % 3]) >= 0
threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
for t in threads: t.start()
for t in threads: t.join()
result = launches()
''')
    assert sum("small_combine" in k for k, *_ in got) == 16
    for i, (kernel, _, _, thread) in enumerate(got):
        if "small_combine" in kernel:
            assert "gemm_kernel" in got[i - 1][0] and got[i - 1][3] == thread, got[i - 1:i + 1]
        elif "fill_zero" in kernel:
            assert "fill_zero" not in got[i + 1][0] and got[i + 1][3] == thread, got[i:i + 2]


# E, H, I, T, topk: batches of full tiles with smaller ones for the rest
LARGE = [(32, 2048, 704, 16384, 6), (30, 2048, 704, 8192, 4), (128, 4096, 1536, 4096, 8),
         (1024, 512, 128, 16384, 8), (1024, 4096, 768, 32768, 8)]


def test_workgroups_of_large_batches(recorder):
    """One workgroup per CU for the up-projection's GEMM, and at most two more
    per CU for the stage's: none is started to find out that there is nothing
    for it to do."""
    got = launch_recorder.run(recorder, f'''
result = []
for E, H, I, T, k in {LARGE}:
    assert call("gemm1", T, H, I, E, k) == 0
    assert call("combine", T, H, I, E, k) == 0
    result.append(launches())
''')
    for shape, calls in zip(LARGE, got):
        calls = [c for c in calls if "fill_zero" not in c[0]]
        assert ["mixed_gemm" in c[0] for c in calls] == [True, True, False], shape
        assert calls[0][1] == 256, (shape, calls[0])
        assert 256 < calls[1][1] <= 3 * 256, (shape, calls[1])


# E, H, I, T, topk and which tiles they run as: the sizes at each limit of the
# rules, and many experts with few rows
ROUTES = {
    "gemm1": [
        (32, 2048, 704, 64, 6, "small"), (64, 2048, 704, 64, 6, "small"), (96, 2048, 704, 64, 6, "small"),
        (128, 2048, 704, 64, 6, "mixed"), (1024, 2048, 768, 64, 8, "mixed"), (8, 4096, 14336, 8, 2, "mixed"),
        # one round of full tiles: more than two small tiles per CU, a longer reduction
        (32, 2048, 704, 650, 6, "small"), (32, 2048, 704, 700, 6, "mixed"), (32, 2048, 704, 1300, 6, "mixed"),
        (30, 2048, 704, 1024, 4, "small"), (30, 2048, 704, 1300, 4, "mixed"), (32, 1024, 512, 1300, 8, "small"),
        (32, 2048, 704, 1600, 6, "small"), (32, 2048, 704, 8192, 6, "mixed"), (11, 1352, 336, 8192, 3, "small"),
    ],
    "combine": [
        (32, 2048, 704, 64, 6, "small"), (128, 2048, 256, 256, 8, "small"), (256, 1024, 256, 512, 8, "small"),
        (96, 4096, 1536, 192, 8, "small"), (128, 4096, 1536, 256, 8, "mixed"), (512, 512, 128, 1024, 8, "mixed"),
        (128, 2048, 256, 2048, 8, "small"), (128, 2048, 256, 2056, 8, "mixed"),
        (30, 2048, 704, 4096, 4, "small"), (32, 2048, 704, 4096, 6, "mixed"), (8, 1024, 512, 8192, 2, "small"),
    ],
}


@pytest.mark.parametrize("op", list(ROUTES))
def test_tiles_by_batch(recorder, op):
    """The rule that chooses between small tiles and full ones counts what both
    would run: it does not turn to full tiles because near-empty experts are
    many, nor to small ones where one round of full tiles is faster."""
    shapes = [s[:5] for s in ROUTES[op]]
    got = launch_recorder.run(recorder, f'''
result = []
for E, H, I, T, k in {shapes}:
    assert call("{op}", T, H, I, E, k) >= 0
    result.append([c[0] for c in launches() if "fill_zero" not in c[0]][0])
''')
    assert [g.split("_gemm_kernel")[0] for g in got] == [s[5] for s in ROUTES[op]], got


def test_fixed_partition_by_environment(recorder):
    """MOE_GEMM2_SELECTOR=0: a call that leaves the choice to the library runs
    with eight dedicated consumers, in every mode; explicit counts win."""
    got = launch_recorder.run(recorder, '''
result = []
for op in ("combine", "noalloc", "layer"):
    for C in (-1, 0, 5):
        for mode in ((0, 1, 2) if op != "layer" else (0,)):
            used = call(op, T=300, H=512, I=64, E=8, topk=2, C=C, mode=mode)
            last = launches()[-1]
            result.append([C, used, last[0], last[1]])
''', MOE_GEMM2_SELECTOR="0")
    for C, used, kernel, grid in got:
        assert used == (8 if C < 0 else C)
        if C == 0:
            assert "small_combine" in kernel
        else:   # 256 CUs, one workgroup each
            assert "moe_gemm2_fused" in kernel and grid == 256


@pytest.mark.parametrize("limit,persistent", [("1", True), ("3999999", True), ("4000000", False),
                                              ("100000000", False)])
def test_wait_limit_by_environment(recorder, limit, persistent):
    """MOE_GEMM2_SPIN_LIMIT bounds the persistent kernel's waits: a limit below
    the built-in one makes the calls without dedicated consumers take it too; one
    that is not leaves them to the launches that never wait."""
    got = launch_recorder.run(recorder, '''
assert call("combine", T=300, H=512, I=64, E=8, topk=2, C=0) == 0
result = launches()[-1][0]
''', MOE_GEMM2_SPIN_LIMIT=limit)
    assert ("moe_gemm2_fused" in got) == persistent, got


TILE_NAMES = {"SmallTile<64, 64, 4, 2, 4, 64>": "64x64", "SmallTile<64, 128, 8, 4, 3, 64>": "64x128 deep",
              "SmallTile<64, 128, 8, 4, 2, 64>": "64x128", "SmallTile<128, 128, 8, 4, 2, 64>": "128x128",
              "SmallTile<128, 256, 8, 4, 3, 32>": "128x256"}


def test_gpu_cases_run_as_the_tiles_they_name(recorder):
    """The GPU tests of the launches without dedicated consumers reach every kind
    of tile, each case the one it is for."""
    import test_gpu_small_batch as cases
    want, calls = [], []
    for name, make in cases.CASES.items():
        w = make()
        calls.append(["combine", w.T, w.H, w.I, w.E, w.topk, w.L, w.Mtot])
        want.append(cases.TILES[name])
    for name, (E, H, I, T, k) in cases.UP.items():
        calls.append(["gemm1", T, H, I, E, k, 1, T * k])
        want.append(cases.UP_TILES[name])
    for E, H, I, rows_of, _, _ in cases.LARGE.values():
        rows = sum(rows_of(e) for e in range(E))
        calls.append(["combine", -(-rows // 4), H, I, E, 4, 1, rows])
        want.append("full")
    for E, N, H, rows_of in cases.UP_LARGE.values():
        rows = sum(rows_of(e) for e in range(E))
        calls.append(["gemm1", -(-rows // 4), H, N // 2, E, 4, 1, rows])
        want.append("full")
    got = launch_recorder.run(recorder, f'''
result = []
for op, T, H, I, E, k, L_, rows in {calls}:
    assert call(op, T, H, I, E, k, splits=L_, rows=rows) >= 0
    result.append([c[0] for c in launches() if "fill_zero" not in c[0]][0])
''')
    kinds = ["full" if "mixed" in g else TILE_NAMES[g[g.index("<") + 1:g.index(">") + 1]] for g in got]
    assert kinds == want, [x for x in zip(calls, kinds, want) if x[1] != x[2]]
    for up in (False, True):
        assert {k for k, c in zip(kinds, calls) if (c[0] == "gemm1") == up} == {*TILE_NAMES.values(), "full"}
