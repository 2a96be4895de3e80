"""GPU: kernels and launch shapes that only some sizes, rank counts or alignments take, each at the edges
of its range, against the oracle bit for bit (NaN results: NaN on both sides)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_bitwise, assert_bitwise_nan_aware, to_dev, to_host
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
