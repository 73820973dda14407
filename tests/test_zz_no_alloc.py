"""The allocation-free entry point (quick_w4a16_gemm_noalloc) through the C
ABI against quick_w4a16_gemm_ex with the same automatic plan: bit-identical
outputs, and within tolerance of the oracle, on two calls in a row (the
second with a smaller input) for every kind of launch that uses a workspace
(split-K partial sums, stream-K partial tiles, the sliced kernel's partial
columns, the wave-split form's K slices with arrival counters and with the
reduction pass) and one that uses none.  The rules run the first two kinds on
none of these sizes: a tune table names them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_10076_amd as Q
from gpu_util import TOL, Packed, from_dev_y, rand_case, rel_err, say, to_dev_x

pytestmark = pytest.mark.gpu

# (K, N, M first call, M second call, tune table entry, launch)
CASES = [
    (4096, 4096, 64, 40, "2 4 32 16", "tiled split-K"),       # fp32 partials + reduction
    (6144, 16384, 256, 200, "3 0 128 32", "stream-K"),        # arrival counters + partial tiles
    (4096, 8192, 16, 12, None, "sliced"),                     # several K slices
    (11008, 1040, 97, 90, None, "wave-split 2 slices"),       # arrival counters
    (11008, 528, 32, 24, None, "wave-split pass"),            # fp32 partials + reduction
    (1024, 272, 3, 1, None, "stream"),                        # no workspace
]


@pytest.fixture(autouse=True)
def no_tune_table():
    Q.tune_table_clear()
    yield
    Q.tune_table_clear()


def _tune(tmp_path, entry, *shapes):
    if entry:
        t = tmp_path / "t.txt"
        t.write_text("quick-tune 1\n" + "".join("%d %d %d %s\n" % (M, N, K, entry) for M, N, K in shapes))
        Q.tune_table_load(str(t))


def _kind(p):
    if p["variant"] == 0:
        return "wave-split pass" if p["launches"] == 2 else "wave-split %d slices" % p["split_k"]
    if p["variant"] == Q.VARIANT_TILED:
        return "tiled split-K" if p["launches"] == 2 else "tiled"
    return {Q.VARIANT_STREAM: "stream", Q.VARIANT_STREAMK: "stream-K", Q.VARIANT_KSTREAM: "sliced"}[p["variant"]]


@pytest.mark.parametrize("K,N,M1,M2,entry,kind", CASES)
def test_noalloc_matches_ex_on_consecutive_calls(tmp_path, K, N, M1, M2, entry, kind):
    _tune(tmp_path, entry, (M1, N, K), (M2, N, K))
    x, q, z, s = rand_case(K + N + M1, M1, K, N)
    p = Packed(q, z, s)
    for M in (M1, M2):
        plan = Q.launch_plan(M, N, K)
        need = Q.workspace_bytes(M, N, K)
        say("noalloc K=%d N=%d M=%d plan=%s workspace=%d" % (K, N, M, plan, need))
        assert _kind(plan) == kind and (need > 0) == (kind != "stream")
        assert need <= Q.SCRATCH_BYTES
        xd = to_dev_x(x[:M])
        y_ex = torch.empty((M, N), dtype=torch.float16, device="cuda")
        ws = torch.zeros(max(need, Q.WS_COUNTER_BYTES) // 4 + 4, dtype=torch.int32, device="cuda")
        Q.w4a16_gemm(xd, p.dw, p.ds, p.dz, N, y=y_ex, workspace=ws)
        y_na = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        Q.w4a16_gemm_noalloc(xd, p.dw, p.ds, p.dz, N, y_na)
        torch.cuda.synchronize()
        a, b = from_dev_y(y_na), from_dev_y(y_ex)
        assert int(ws[:Q.WS_COUNTER_BYTES // 4].abs().sum().item()) == 0
        assert np.array_equal(a, b), "noalloc differs from the _ex call at %d entries" % int((a != b).sum())
        # the oracle on every row and one column of every n-tile (rotating position)
        t = np.arange(N // 16)
        cols = 16 * t + (t % 16)
        assert rel_err(a[:, cols], oracle.gemm(x[:M], q, z, s, cols=cols)) <= TOL


@pytest.mark.parametrize("K,N,M,entry,kind", [
    (6144, 16384, 256, "3 0 128 32", "stream-K"),           # counters and partial tiles in the scratch array
    (11008, 1040, 97, None, "wave-split 2 slices"),         # counters and partial sums
    (11008, 528, 32, None, "wave-split pass")])             # partial sums
def test_noalloc_repeated_calls_and_capture(tmp_path, K, N, M, entry, kind):
    """The scratch counters are left zero: ten calls in a row give the same
    bits, also when the calls are captured in a graph and replayed."""
    _tune(tmp_path, entry, (M, N, K))
    assert _kind(Q.launch_plan(M, N, K)) == kind
    x, q, z, s = rand_case(91, M, K, N)
    p = Packed(q, z, s)
    xd = to_dev_x(x)
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    Q.w4a16_gemm_noalloc(xd, p.dw, p.ds, p.dz, N, y)
    torch.cuda.synchronize()
    first = y.clone()
    for _ in range(10):
        Q.w4a16_gemm_noalloc(xd, p.dw, p.ds, p.dz, N, y)
    torch.cuda.synchronize()
    assert torch.equal(y, first)
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):          # nothing to allocate: captures on a fresh stream
        Q.w4a16_gemm_noalloc(xd, p.dw, p.ds, p.dz, N, y)
    for _ in range(3):
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, first)
        Q.w4a16_gemm_noalloc(xd[:7], p.dw, p.ds, p.dz, N, torch.empty((7, N), dtype=torch.float16, device="cuda"))
        torch.cuda.synchronize()
