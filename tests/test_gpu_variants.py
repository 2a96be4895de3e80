"""GPU: kernels and launch shapes that only some sizes, rank counts or alignments take, each at the edges
of its range, against the oracle bit for bit (NaN results: NaN on both sides)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_bitwise, assert_bitwise_nan_aware, run_combine, to_dev, to_host
from test_zz_no_alloc import _check_case as check_routed
from paper_2608_00867_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GUARD = 64


@pytest.fixture(scope="module")
def nuna():
    from paper_2608_00867_amd import nuna as n
    n.init()
    return n


@pytest.fixture(autouse=True)
def _free():
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _guarded(n, dtype):
    whole = torch.empty(n + 2 * GUARD, dtype=dtype, device="cuda")
    whole.view(torch.int16 if dtype == torch.bfloat16 else torch.int32).fill_(0x5A5A)
    return whole[GUARD:GUARD + n], whole


def _intact(whole, n, what):
    w = whole.view(torch.int16 if whole.dtype == torch.bfloat16 else torch.int32).cpu().numpy()
    assert np.all(w[:GUARD] == 0x5A5A) and np.all(w[GUARD + n:] == 0x5A5A), f"{what}: write outside the output"


def _values(P, n, dtype, seed):
    return wl.normal_bf16(P, n, seed) if dtype == "bf16" else wl.normal_f32(P, n, seed)


def _run(call, x, n_out, what):
    ins = [to_dev(a) for a in x]
    pairs = [_guarded(n_out, ins[0].dtype) for _ in x]
    call(ins, [p[0] for p in pairs])
    torch.cuda.synchronize()
    for _, whole in pairs:
        _intact(whole, n_out, what)
    return [to_host(o) for o, _ in pairs]


# ---------------------------------------------------------------- fp32 -> bf16 narrowing

def test_bf16_narrowing_of_every_high_half(nuna):
    """hi + lo over every bf16 pattern hi and a lo below its last place: ties, values just off a tie,
    denormals, overflow to infinity, infinities and NaN, in even and odd lanes of a vector."""
    hi = np.arange(1 << 16, dtype=np.uint16)
    half = (hi.astype(np.uint32) << 16).view(np.float32)
    with np.errstate(all="ignore"):
        for scale in (2.0 ** -9, 1.5 * 2.0 ** -9, -(2.0 ** -9), 2.0 ** -10):
            lo = wl.f32_to_bf16_bits((half * np.float32(scale)).astype(np.float32))
            for shift in (0, 1):
                x = [np.roll(hi, shift), np.roll(lo, shift)]
                ref = oracle.allreduce(x)
                outs = nuna.allreduce([to_dev(a) for a in x])
                torch.cuda.synchronize()
                assert_bitwise_nan_aware(to_host(outs[0]), ref[0], f"scale {scale} shift {shift}")


# ---------------------------------------------------------------- all-reduce launch shapes

SHAPE_EDGES = [(2, "f32", 16), (2, "bf16", 13), (2, "bf16", 128), (4, "f32", 13), (4, "bf16", 13), (4, "bf16", 20),
               (8, "f32", 9), (8, "f32", 13), (8, "f32", 26), (8, "f32", 33), (8, "bf16", 9), (8, "bf16", 33),
               (16, "f32", 5), (16, "f32", 9), (16, "f32", 15), (16, "bf16", 9), (16, "bf16", 13), (16, "bf16", 20)]


@pytest.mark.parametrize("P,dtype,quarter", SHAPE_EDGES)
def test_allreduce_shape_edges(nuna, P, dtype, quarter):
    """One vector below each size where the launch shape changes, and above it by a vector and a tail."""
    es = 2 if dtype == "bf16" else 4
    at = quarter * (1 << 18) // es
    for n in (at - 16 // es, at + 16 // es + 3):
        what = f"P={P} {dtype} n={n}"
        x = _values(P, n, dtype, 17 * quarter + P)
        ref = oracle.allreduce(x)
        got = _run(lambda i, o: nuna.allreduce(i, o, algo="one_shot"), x, n, what)
        for d in (0, P // 2, P - 1):
            assert_bitwise(got[d], ref[d], f"{what} rank {d}")


# ---------------------------------------------------------------- rank counts without a kernel of their own

@pytest.mark.parametrize("P", [1, 3, 5, 6, 7, 9, 12, 15])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_run_time_rank_counts(nuna, P, dtype):
    """All-reduce, reduce-scatter and all-gather of every register bucket of run-time rank counts (up to 4,
    8 and 16), one vector, a chunk and a vector, and sizes of the shape rows; in place too."""
    es = 2 if dtype == "bf16" else 4
    lanes = 16 // es
    for n in (lanes, 1024 * lanes + lanes + 1, 5 * (1 << 16) * lanes + 3, 7 * (1 << 17) * lanes):
        what = f"P={P} {dtype} n={n}"
        x = _values(P, n, dtype, 31 * P + n % 97)
        ref = oracle.allreduce(x)
        got = _run(nuna.allreduce, x, n, what)
        bufs = [to_dev(a) for a in x]
        nuna.allreduce(bufs, bufs, algo="one_shot")
        torch.cuda.synchronize()
        for d in {0, P // 2, P - 1}:
            assert_bitwise(got[d], ref[d], f"{what} rank {d}")
            assert_bitwise(to_host(bufs[d]), ref[d], f"{what} in place rank {d}")
    for m in (lanes, 129 * lanes, ((1 << 17) // P + 5) * lanes, ((5 << 18) // P + 1) * lanes):
        what = f"P={P} {dtype} m={m}"
        x = _values(P, P * m, dtype, 37 * P + m % 89)
        ref = oracle.reduce_scatter(x)
        got = _run(nuna.reduce_scatter, x, m, "RS " + what)
        src = [a[:m].copy() for a in x]
        ref_g = oracle.all_gather(src)
        got_g = _run(nuna.all_gather, src, P * m, "AG " + what)
        bufs = [torch.zeros(P * m, dtype=to_dev(src[0]).dtype, device="cuda") for _ in range(P)]
        for r in range(P):
            bufs[r][r * m:(r + 1) * m].copy_(to_dev(src[r]))
        nuna.all_gather([bufs[r][r * m:(r + 1) * m] for r in range(P)], bufs)
        torch.cuda.synchronize()
        for d in {0, P // 2, P - 1}:
            assert_bitwise(got[d], ref[d], f"RS {what} rank {d}")
            assert_bitwise(got_g[d], ref_g[d], f"AG {what} rank {d}")
            assert_bitwise(to_host(bufs[d]), ref_g[d], f"AG {what} in place rank {d}")


RS_EDGES = [(2, 32), (4, 3), (4, 16), (4, 32), (8, 1), (8, 7), (8, 16), (8, 32), (12, 18), (12, 30), (16, 2), (16, 5),
            (16, 10), (16, 14), (16, 18), (16, 28)]


@pytest.mark.parametrize("P,quarter", RS_EDGES)
def test_reduce_scatter_shape_edges(nuna, P, quarter):
    """fp32, shards one vector below and above each size where the launch shape changes."""
    at = quarter * (1 << 14) // P  # vectors per shard
    for mv in (at - 1, at + 1):
        x = wl.normal_f32(P, P * mv * 4, 41 * quarter + P)
        ref = oracle.reduce_scatter(x)
        got = _run(nuna.reduce_scatter, x, mv * 4, f"P={P} mv={mv}")
        for r in (0, P - 1):
            assert_bitwise(got[r], ref[r], f"P={P} mv={mv} rank {r}")


# ---------------------------------------------------------------- ragged shards

@pytest.mark.parametrize("P", [2, 3, 5, 8, 11, 16, 20, 64])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_ragged_shards(nuna, P, dtype):
    """Shards of every remainder of a vector, below one vector, around chunk edges and at several vectors
    per thread: reduce-scatter, all-gather, and the two-shot in place (whose shards begin at any element)."""
    lanes = 8 if dtype == "bf16" else 4
    big = (1 << 19) // P // (4 if P > 16 else 1)
    big = max(big, 3 * (1 << 16) // P)
    sizes = [1, 2, lanes - 1, lanes + 1] + [64 * lanes + e for e in range(1, lanes)] + \
        [256 * lanes - 1, 256 * lanes + 1, big * lanes // 4 + 3, big * lanes // 2 + 1]
    for k, m in enumerate(sizes):
        what = f"P={P} {dtype} m={m}"
        x = _values(P, P * m, dtype, 43 * P + k)
        ref = oracle.reduce_scatter(x)
        got = _run(nuna.reduce_scatter, x, m, "RS " + what)
        src = [a[:m].copy() for a in x]
        ref_g = oracle.all_gather(src)
        got_g = _run(nuna.all_gather, src, P * m, "AG " + what)
        ref_a = oracle.allreduce(x)
        bufs = [to_dev(a) for a in x]
        nuna.allreduce(bufs, bufs, algo="two_shot_two_kernels")
        torch.cuda.synchronize()
        for d in range(P):
            assert_bitwise(got[d], ref[d], f"RS {what} rank {d}")
        for d in {0, P // 2, P - 1}:
            assert_bitwise(got_g[d], ref_g[d], f"AG {what} rank {d}")
            assert_bitwise(to_host(bufs[d]), ref_a[d], f"two-shot {what} rank {d}")


@pytest.mark.parametrize("cap", [1, 3, 40])
def test_ragged_shards_under_a_workgroup_cap(nuna, cap):
    """A capped launch walks on over chunks and shards, with no more workgroups than the cap."""
    P, m = 6, 5003
    x = _values(P, P * m, "bf16", 5)
    src = [a[:m].copy() for a in x]
    nuna.set_max_workgroups(cap)
    try:
        got = _run(nuna.reduce_scatter, x, m, "RS")
        assert nuna.last_launch()["grid"] <= cap
        got_g = _run(nuna.all_gather, src, P * m, "AG")
        assert nuna.last_launch()["grid"] <= cap
    finally:
        nuna.set_max_workgroups(0)
    ref, ref_g = oracle.reduce_scatter(x), oracle.all_gather(src)
    for d in range(P):
        assert_bitwise(got[d], ref[d], f"RS rank {d}")
        assert_bitwise(got_g[d], ref_g[d], f"AG rank {d}")


@pytest.mark.parametrize("H", [8, 2048, 2056, 4088, 4096, 4104])
@pytest.mark.parametrize("P,T,k,E", [(1, 260, 1, 1), (3, 87, 3, 12), (4, 130, 4, 32), (8, 33, 8, 64), (7, 150, 5, 28),
                                     (9, 40, 4, 36), (16, 70, 8, 64), (17, 16, 8, 68)])
def test_routed_row_lengths(nuna, P, T, k, E, H):
    """The routed and the layout-driven dispatch at the row lengths where their threads change (256 and 512
    vectors) and around them; rank counts at the edges of the counting kernel's 8, 16 and 64; records of 4, 8 and
    odd words; the last wave of a source partly filled; a receive buffer with no row to spare."""
    for place in ("linear", "xcd"):
        check_routed(nuna, P, T, k, E, H, 31 * P + H, place, cap_extra=8 if place == "xcd" else 0)


@pytest.mark.parametrize("grid", [5, 8, 61])
def test_routed_row_lengths_under_a_workgroup_cap(nuna, grid):
    with nuna.tunables(NUNA_MAX_GRID=grid):
        for P, T, k, E, H in ((8, 40, 8, 64, 264), (12, 30, 3, 36, 2056), (33, 9, 2, 66, 4104)):
            for place in ("linear", "xcd"):
                check_routed(nuna, P, T, k, E, H, 77 + P, place)


@pytest.mark.parametrize("dtype", [np.uint16, np.float32])
@pytest.mark.parametrize("P,T,k,E", [(9, 5, 4, 36), (16, 3, 8, 64), (33, 4, 8, 66), (8, 6, 8, 64)])
def test_combine_lists_row_lengths(nuna, P, T, k, E, dtype):
    """The combine from offset lists, one pass per column chunk: rows of one vector, of a workgroup's 256 and one
    more or less, of several chunks with a short last one; plain and weighted; a fixed chunk count of several
    passes.  8 ranks: the lists by the tunable."""
    topk = wl.moe_routing(P, T, k, E, 5 * P)
    lanes = 8 if dtype == np.uint16 else 4
    lay = nuna.A2ALayout(topk, E)
    rows = [int(r) for r in lay.recv_rows()]
    lay.close()
    weights = wl.gate_weights(topk, E, 9)
    for vecs, tune in ((1, {}), (255, {}), (256, {}), (257, {}), (700, {}), (1025, {}), (700, {"NUNA_COMBINE_CHUNKS": 1})):
        H = vecs * lanes
        y = wl.result_rows(rows, H, dtype, vecs)
        for w in (None, weights):
            want = oracle.combine(y, topk, E, w)
            with nuna.tunables(**dict(tune, NUNA_COMBINE_LISTS=1)):
                got = run_combine(nuna, y, topk, E, "xcd", weights=w)
            for s in range(P):
                assert_bitwise(got[s], want[s], f"combine lists P={P} vecs={vecs} {tune} w={w is not None} rank {s}")
