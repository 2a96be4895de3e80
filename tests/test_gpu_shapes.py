"""GPU: the launch shapes that a workgroup cap, the split and the two-shot all-reduce and the rank-count rules
choose, by the launch record, with results against the oracle bit for bit; and two chunk forms whose loads have
to be in flight together, by their time beside that of whole chunks."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_bitwise, run_combine, to_dev, to_host
from test_gpu_parity import run_allreduce
from paper_2608_00867_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MIB = 1 << 20
ES = {"bf16": 2, "f32": 4}


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


def _values(P, n, dtype, seed):
    return wl.normal_bf16(P, n, seed) if dtype == "bf16" else wl.normal_f32(P, n, seed)


def _allreduce(nuna, P, dtype, n, what, algo="one_shot", check=True):
    """The launch record of one all-reduce of n elements per rank, checked on three ranks."""
    x = _values(P, n, dtype, 7 * P + n % 101) if check else None
    if check:
        ins = [to_dev(a) for a in x]
    else:
        ins = [torch.zeros(n, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
               for _ in range(P)]
    outs = nuna.allreduce(ins, algo=algo)
    rec = nuna.last_launch()
    torch.cuda.synchronize()
    if check:
        ref = oracle.allreduce(x)
        for d in {0, P // 2, P - 1}:
            assert_bitwise(to_host(outs[d]), ref[d], f"{what} rank {d}")
    return rec


def _us(call, n=60):
    """Device time of one call, from the fastest of several replays of a graph of n."""
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(n):
            call()
    best = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        torch.cuda.synchronize()
        best.append(a.elapsed_time(b) * 1e3 / n)
    return min(best)


# ---------------------------------------------------------------- loads in flight together

@pytest.mark.parametrize("P,chunks", [(6, 220), (9, 200), (12, 190), (14, 202), (15, 108)])
def test_a_partial_chunk_takes_no_longer_than_a_whole_one(nuna, P, chunks):
    """Run-time rank counts, bf16, 256 threads with one vector: a message that ends in a partial chunk runs in
    the time of one that does not.  With its ranks loaded one after another the last workgroup alone took as long
    again as the whole launch (1.3-2.0 times the time of whole chunks); loaded together, within 6 %."""
    def time(n):
        ins = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(P)]
        outs = [torch.empty_like(t) for t in ins]
        call = nuna.prepare_allreduce(ins, outs)
        call()
        assert nuna.last_launch()["threads"] == 256 and nuna.last_launch()["kernels"] == "k_allreduce_direct"
        return _us(lambda: call(torch.cuda.current_stream().cuda_stream))

    whole, partial = time(chunks * 2048), time(chunks * 2048 - 1024)
    assert partial < 1.2 * whole, (partial, whole)


def test_partial_chunks_of_ragged_shards(nuna):
    """The same for 16 ranks of bf16 and shards of no whole vectors: 129 vectors and a rest per shard against 128
    and a rest (4.04 against 2.82 us with the ranks one after another, 2.97 against 2.77 together)."""
    def time(m):
        ins = [torch.zeros(16 * m, dtype=torch.bfloat16, device="cuda") for _ in range(16)]
        outs = [torch.empty(m, dtype=torch.bfloat16, device="cuda") for _ in range(16)]
        return _us(lambda: nuna.reduce_scatter(ins, outs))

    whole, partial = time(1031), time(1033)
    assert partial < 1.25 * whole, (partial, whole)


@pytest.mark.parametrize("P", [3, 7, 13])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_messages_below_a_vector_and_partial_chunks(nuna, P, dtype):
    """Run-time rank counts: less than one vector (a tail alone), one vector, and partial chunks whose lanes past
    the end load the last vector; in place, guard bands by the caller's neighbours."""
    lanes = 16 // ES[dtype]
    for n in (1, lanes - 1, lanes, lanes + 1, 255 * lanes, 257 * lanes + 1, 70001):
        x = _values(P, n, dtype, 3 * P + n)
        ref = oracle.allreduce(x)
        with nuna.tunables(NUNA_LPR_MIN_RANKS=65):
            got = run_allreduce(nuna, x, "one_shot", "xcd")
            bufs = [to_dev(a) for a in x]
            nuna.allreduce(bufs, bufs, algo="one_shot")
            torch.cuda.synchronize()
        for d in range(P):
            assert_bitwise(got[d], ref[d], f"P={P} {dtype} n={n} rank {d}")
            assert_bitwise(to_host(bufs[d]), ref[d], f"P={P} {dtype} n={n} in place rank {d}")


@pytest.mark.parametrize("P", [17, 24, 33, 64])
def test_tails_of_many_ranks(nuna, P):
    """Elements after the last vector, summed 16 ranks at a time: one round and a rest, and four whole rounds."""
    for dtype in ("bf16", "f32"):
        for n in (3, 16 * (16 // ES[dtype]) + 1, 5003):
            _allreduce(nuna, P, dtype, n, f"tail P={P} {dtype} n={n}")


# ---------------------------------------------------------------- shapes under a workgroup cap

def test_capped_all_reduce_and_reduce_scatter_shapes(nuna):
    """A capped launch loops over its items in few workgroups: they are of 256 threads (or hold 4 and more vectors),
    not the one-wave workgroups that fill the chip otherwise, and 9 to 15 ranks leave the tile kernel."""
    cases = [(6, "bf16", 3 * MIB // 4, (256, 1)), (6, "f32", 3 * MIB // 8, (256, 1)), (8, "f32", 9 * MIB // 16, (256, 1)),
             (8, "bf16", 2 * MIB, (256, 2)), (16, "bf16", 9 * MIB // 8, (256, 1)), (2, "f32", MIB, (128, 4)),
             (12, "f32", 3 * MIB // 2, (128, 4)), (8, "bf16", 4 * MIB, (256, 8))]
    nuna.set_max_workgroups(64)
    try:
        for P, dtype, n, shape in cases:
            rec = _allreduce(nuna, P, dtype, n + 3, f"cap AR P={P} {dtype} n={n}")
            assert (rec["threads"], rec["vectors_per_thread"]) == shape and rec["grid"] <= 64, (P, dtype, n, rec)
        rec = _allreduce(nuna, 12, "bf16", MIB // 8, "cap AR 12 ranks")
        assert rec["kernels"] == "k_allreduce_direct" and rec["threads"] == 256 and rec["grid"] <= 64, rec
        for P, dtype, m in ((4, "bf16", 3 * MIB // 16), (6, "f32", MIB // 16), (8, "bf16", MIB // 16),
                            (8, "f32", MIB // 64), (12, "bf16", MIB // 16), (16, "f32", MIB // 128)):
            x = _values(P, P * m, dtype, 11 * P)
            outs = nuna.reduce_scatter([to_dev(a) for a in x])
            rec = nuna.last_launch()
            torch.cuda.synchronize()
            ref = oracle.reduce_scatter(x)
            for r in (0, P - 1):
                assert_bitwise(to_host(outs[r]), ref[r], f"cap RS P={P} {dtype} rank {r}")
            assert rec["threads"] == 256 and rec["grid"] <= 64, (P, dtype, m, rec)
    finally:
        nuna.set_max_workgroups(0)
    assert _allreduce(nuna, 6, "bf16", 3 * MIB // 4, "uncapped")["threads"] == 64


def test_capped_moe_shapes(nuna):
    """Short rows under a cap keep 256 threads, and the combine from lists 2 vectors per thread."""
    P, T, k, E, H = 16, 40, 4, 64, 2048
    topk = wl.moe_routing(P, T, k, E, 5)
    send_np = wl.moe_rows(P, T, H, 6)
    ref = oracle.all_to_all(send_np, topk, E)
    back = oracle.combine(ref, topk, E, None)
    lay = nuna.A2ALayout(topk, E).upload()
    rows = [int(v) for v in lay.recv_rows()]
    recv = [torch.zeros((max(rows), H), dtype=torch.bfloat16, device="cuda") for _ in range(P)]
    send = [to_dev(a.reshape(-1)).view(T, H) for a in send_np]
    topk_dev = torch.from_numpy(np.ascontiguousarray(topk)).cuda()
    counts = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    for cap, threads in ((40, 256), (0, 64)):
        nuna.set_max_workgroups(cap)
        try:
            nuna.all_to_all(send, recv, lay, placement="linear")
            assert nuna.last_launch()["threads"] == threads, nuna.last_launch()
            nuna.all_to_all_routed(send, recv, topk_dev, E, counts, placement="linear")
            assert nuna.last_launch()["threads"] == threads, nuna.last_launch()
            torch.cuda.synchronize()
            for d in range(P):
                assert_bitwise(to_host(recv[d])[:rows[d]], ref[d], f"cap {cap} dispatch rank {d}")
            got = run_combine(nuna, ref, topk, E, "linear")
            assert nuna.last_launch()["vectors_per_thread"] == (2 if cap else 1), nuna.last_launch()
        finally:
            nuna.set_max_workgroups(0)
        for s in range(P):
            assert_bitwise(got[s], back[s], f"cap {cap} combine rank {s}")
    lay.close()


# ---------------------------------------------------------------- split and two-shot shapes

@pytest.mark.parametrize("P,dtype,mib,shape", [(8, "bf16", 3.5, (256, 1)), (8, "bf16", 7, (128, 4)), (8, "f32", 7, (128, 4)),
                                               (3, "bf16", 3, (256, 1)), (16, "bf16", 3.5, (256, 1)),
                                               (16, "f32", 2.5, (256, 1)), (6, "f32", 8, (128, 4)), (6, "bf16", 8, (256, 4)),
                                               (12, "bf16", 3, (256, 1)), (12, "bf16", 6, (128, 2)), (2, "bf16", 4, (64, 8)),
                                               (2, "bf16", 8, (128, 4))])
def test_split_all_reduce_shapes(nuna, P, dtype, mib, shape):
    """The split all-reduce has the shared rule's shapes, not the one-shot's, except where those measured faster."""
    rec = _allreduce(nuna, P, dtype, int(mib * MIB) // ES[dtype], f"split P={P} {dtype} {mib} MiB", algo="one_shot_split",
                     check=mib <= 4)
    assert (rec["threads"], rec["vectors_per_thread"]) == shape, rec


@pytest.mark.parametrize("P,dtype,mib,shape", [(2, "f32", 4, (128, 4)), (2, "f32", 8, (128, 4)), (2, "f32", 8.25, (64, 8)),
                                               (4, "bf16", 3.25, (256, 1)), (4, "bf16", 3.5, (256, 2)),
                                               (8, "bf16", 16, (256, 8))])
def test_fused_two_shot_shapes(nuna, P, dtype, mib, shape):
    rec = _allreduce(nuna, P, dtype, int(mib * MIB) // ES[dtype], f"two-shot P={P} {dtype} {mib} MiB", algo="two_shot",
                     check=mib <= 4)
    assert rec["kernels"] == "k_two_shot_direct" and (rec["threads"], rec["vectors_per_thread"]) == shape, rec


@pytest.mark.parametrize("P,n", [(6, 6 * 131072), (6, 6 * 87384), (16, MIB // 2)])
def test_two_shot_of_two_kernels_at_2_to_4_mib(nuna, P, n):
    """The sizes whose reduce-scatter phase is cut as its all-gather phase is."""
    for dtype in ("bf16", "f32"):
        _allreduce(nuna, P, dtype, n * 4 // ES[dtype], f"two kernels P={P} {dtype}", algo="two_shot_two_kernels")


@pytest.mark.parametrize("P,dtype,quarters,shape", [(16, "bf16", 8, (256, 2)), (16, "bf16", 8.2, (256, 1)),
                                                    (16, "f32", 8.2, (256, 1)), (16, "f32", 9, (64, 4)),
                                                    (11, "f32", 26, (128, 4)), (11, "f32", 32, (256, 4)),
                                                    (11, "f32", 33, (128, 4)), (11, "bf16", 26, (128, 2)),
                                                    (7, "f32", 4.6, (64, 1)), (6, "f32", 11, (64, 1)),
                                                    (7, "f32", 10, (64, 1)), (7, "f32", 11, (128, 2)),
                                                    (7, "f32", 13.5, (256, 1)), (6, "f32", 12, (256, 1)),
                                                    (7, "bf16", 8, (256, 1)),
                                                    (2, "bf16", 13, (256, 1)), (2, "bf16", 15, (64, 8))])
def test_one_shot_rows(nuna, P, dtype, quarters, shape):
    n = int(quarters * (1 << 18)) // ES[dtype] // 64 * 64 + 3
    rec = _allreduce(nuna, P, dtype, n, f"P={P} {dtype} {quarters}", check=quarters < 16)
    assert (rec["threads"], rec["vectors_per_thread"]) == shape, rec


@pytest.mark.parametrize("quarters,extra,shape", [(17, 0, (64, 4)), (18, 0, (64, 1)), (20, 0, (64, 1)), (20, 1, (64, 4)),
                                                  (22, 0, (64, 1)), (23, 0, (64, 4))])
def test_reduce_scatter_rows_of_fp32(nuna, quarters, extra, shape):
    """8 ranks of fp32 at 4.25 to 5.75 MiB of input: a call of whole vectors, ragged shards, and the phase of the
    two kernels, whose chunk stays the all-gather's."""
    m = quarters * 65536 // 8 + extra
    x = _values(8, 8 * m, "f32", quarters)
    ref = oracle.reduce_scatter(x)
    outs = nuna.reduce_scatter([to_dev(a) for a in x])
    rec = nuna.last_launch()
    assert (rec["threads"], rec["vectors_per_thread"]) == shape, rec
    torch.cuda.synchronize()
    for d in (0, 7):
        assert_bitwise(to_host(outs[d]), ref[d], f"{quarters} quarters + {extra} shard {d}")
    _allreduce(nuna, 8, "f32", 8 * (m & ~3), f"two kernels {quarters}", algo="two_shot_two_kernels")


# ---------------------------------------------------------------- tunables

def test_many_rank_tunable_says_from_where(nuna):
    """9 to 15 ranks run the tile kernel by default and not when the tunable names a higher count, 16 among them, nor
    when the caller fixes the threads or the vectors; 16 ranks run it in each case."""
    n = 64 << 10 >> 1
    assert _allreduce(nuna, 12, "bf16", n, "default")["kernels"] == "k_allreduce_tile_direct"
    for tune, shape in ((dict(NUNA_LPR_MIN_RANKS=16), None), (dict(NUNA_LPR_MIN_RANKS=13), None),
                        (dict(NUNA_VPT=2), (64, 2)), (dict(NUNA_WG_THREADS=128), (128, 1))):
        with nuna.tunables(**tune):
            rec = _allreduce(nuna, 12, "bf16", n, str(tune))
            assert rec["kernels"] == "k_allreduce_direct", (tune, rec)
            assert shape is None or (rec["threads"], rec["vectors_per_thread"]) == shape, (tune, rec)
            assert _allreduce(nuna, 16, "bf16", n, f"16 ranks {tune}")["kernels"] == "k_allreduce_tile_direct"
    with nuna.tunables(NUNA_LPR_MIN_RANKS=12, NUNA_VPT=2):
        assert _allreduce(nuna, 12, "bf16", n, "named")["kernels"] == "k_allreduce_tile_direct"


# ---------------------------------------------------------------- ragged shards

@pytest.mark.parametrize("P", [9, 10, 13, 14, 17, 18])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_ragged_routes(nuna, P, dtype):
    """Shards on either side of the element kernels' ranges, and destination groups that do not divide the ranks."""
    es = ES[dtype]
    for kib in (2, 19, 21, 41, 43, 73):
        m = (kib << 10) // es + 1
        what = f"P={P} {dtype} m={m}"
        x = _values(P, P * m, dtype, 13 * P + kib)
        ref = oracle.reduce_scatter(x)
        outs = nuna.reduce_scatter([to_dev(a) for a in x])
        rs = nuna.last_launch()["kernels"]
        src = [a[:m].copy() for a in x]
        ref_g = oracle.all_gather(src)
        outs_g = nuna.all_gather([to_dev(a) for a in src])
        ag = nuna.last_launch()["kernels"]
        torch.cuda.synchronize()
        for d in range(P):
            assert_bitwise(to_host(outs[d]), ref[d], f"RS {what} rank {d}")
        for d in {0, P // 2, P - 1}:
            assert_bitwise(to_host(outs_g[d]), ref_g[d], f"AG {what} rank {d}")
        low, high = 20, 72 if dtype == "f32" and P <= 12 else 42 if dtype == "f32" and P <= 16 or P <= 12 else 0
        assert ag == ("k_all_gather_elem" if low <= kib < high else "k_all_gather_ragged"), (what, ag)
        elem = P < 16 and P * m <= 1 << 19 or P > 16 and dtype == "bf16" and P * m <= 216 << 10
        assert rs == ("k_reduce_scatter_elem" if elem else "k_reduce_scatter_ragged"), (what, rs)


# ---------------------------------------------------------------- MoE

@pytest.mark.parametrize("dtype,P,T,k,vpt", [("bf16", 16, 40, 1, 2), ("bf16", 16, 40, 8, 1), ("bf16", 9, 20, 1, 1),
                                             ("f32", 16, 40, 8, 2), ("f32", 9, 20, 8, 1)])
def test_combine_of_rows_between_one_and_two_chunks(nuna, dtype, P, T, k, vpt):
    """Rows of 360 vectors from offset lists: one chunk of 2 vectors with few rows per token, else two chunks."""
    E = 8 * P
    H = 360 * (16 // ES[dtype])
    topk = wl.moe_routing(P, T, k, E, 3 * P)
    lay = nuna.A2ALayout(topk, E)
    rows = [int(v) for v in lay.recv_rows()]
    lay.close()
    y = wl.result_rows(rows, H, np.uint16 if dtype == "bf16" else np.float32, 4)
    for w in (None, wl.gate_weights(topk, E, 9)):
        got = run_combine(nuna, y, topk, E, "xcd", weights=w)
        assert nuna.last_launch()["vectors_per_thread"] == vpt, nuna.last_launch()
        want = oracle.combine(y, topk, E, w)
        for s in range(P):
            assert_bitwise(got[s], want[s], f"combine {dtype} P={P} k={k} w={w is not None} rank {s}")


def test_layout_tables_beyond_one_staged_copy(nuna):
    """A layout of more than 16 MiB of tables, which go up one by one: dispatch and combine against the oracle."""
    P, T, k, E, H = 8, 9000, 8, 64, 8
    topk = wl.moe_routing(P, T, k, E, 71)
    lay = nuna.A2ALayout(topk, E).upload()
    rows = [int(v) for v in lay.recv_rows()]
    assert 40 * sum(rows) + 40 * P * T > 16 * MIB
    send_np = wl.moe_rows(P, T, H, 72)
    want = oracle.all_to_all(send_np, topk, E)
    send = [to_dev(a.reshape(-1)).view(T, H) for a in send_np]
    for place in ("linear", "xcd"):
        recv = [torch.zeros((max(rows), H), dtype=torch.bfloat16, device="cuda") for _ in range(P)]
        nuna.all_to_all(send, recv, lay, placement=place)
        out = [torch.zeros((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(P)]
        nuna.all_to_all_combine(recv, out, lay, placement=place)
        torch.cuda.synchronize()
        for d in range(P):
            assert_bitwise(to_host(recv[d])[:rows[d]], want[d], f"dispatch {place} rank {d}")
        back = oracle.combine(want, topk, E, None)
        for s in range(P):
            assert_bitwise(to_host(out[s]), back[s], f"combine {place} rank {s}")
    lay.close()
