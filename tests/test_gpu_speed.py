"""GPU: calls without dedicated consumers take no longer than the persistent
kernel takes for the same call (its role switch, which a traced call runs), on
batches that are far from the usual ones.  The limit is 1.25 times, on medians
of back-to-back calls; what these guard against was a factor of 1.4 to 13."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _calls(E, H, I, rows, topk, token_of):
    import torch

    from paper_2609_07536_amd import binding as B
    counts = np.full(E, rows)
    n, gen = int(counts.sum()), torch.Generator(device="cuda").manual_seed(3)
    T = -(-n // topk)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda").bfloat16()

    x, w2, gate = normal(n, I), normal(E, I, H), torch.rand(n, generator=gen, device="cuda")
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    tid = torch.from_numpy(token_of(np.random.default_rng(4), n, T, topk).astype(np.int32)).cuda()
    wl, _ = B.make_workload(T, H, I, E, topk, 1, rows=n)
    ws = B.Workspace(B.workspace_size(wl))
    out = torch.empty((T, H), device="cuda")
    trace = torch.zeros(B.trace_size(wl) // 8, dtype=torch.int64, device="cuda")

    def call(mode, traced):
        B.combine(x, w2, off, tid, gate, T=T, topk=topk, num_consumers=0, out=out, workspace=ws, mode=mode,
                  trace=trace if traced else None)
        return out
    return call


def _median_us(call, mode, traced):
    import torch
    for _ in range(3):
        call(mode, traced)
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(6):
            call(mode, traced)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / 6)
    return float(np.median(times))


def _spread(rng, n, T, topk):
    return rng.permutation(np.repeat(np.arange(T), topk)[:n])


@pytest.mark.parametrize("E,H,I,rows", [(1024, 1024, 256, 16), (512, 2048, 256, 48),
                                        (1024, 512, 128, 100), (1024, 2048, 256, 1)])
def test_many_experts(gpu_lib, E, H, I, rows):
    call = _calls(E, H, I, rows, 8, _spread)
    persistent, now = _median_us(call, 0, True), _median_us(call, 0, False)
    print(f"E={E} H={H} I={I} rows={rows}: persistent {persistent:.1f} us, two launches {now:.1f} us", flush=True)
    assert now <= 1.25 * persistent


@pytest.mark.parametrize("name", ["one", "few", "half", "late"])
def test_rows_past_topk(gpu_lib, name):
    """The atomic scatter where tokens have more than topk rows: half of all
    rows are one token's or 64 tokens', every second token has twice topk, and
    one token's rows come at the end of every expert."""
    def token_of(rng, n, T, topk):
        tid = _spread(rng, n, T, topk)
        if name == "one":
            tid[rng.permutation(n)[:n // 2]] = 5
        elif name == "few":
            idx = rng.permutation(n)[:n // 2]
            tid[idx] = rng.integers(0, 64, n // 2)
        elif name == "half":
            tid &= ~1
        else:
            tid[n // 16 * np.arange(1, 17)[:, None] - np.arange(1, 200)] = T - 1
        return tid
    call = _calls(16, 1024, 256, 4096, 8, token_of)
    persistent, now = _median_us(call, 1, True), _median_us(call, 1, False)
    print(f"{name}: persistent {persistent:.1f} us, two launches {now:.1f} us", flush=True)
    assert now <= 1.25 * persistent
    want, got = call(1, True).clone(), call(1, False)
    # fp32 sums of up to 32768 terms of about unit size in other orders
    assert (got - want).norm() <= 1e-5 * want.norm()
