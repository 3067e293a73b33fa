"""nm_project with scale groups of several rows in one launch: the workgroups of a group exchange their maxima, or, out of patience,
read the rest of the group themselves; under capture and in place the call takes its other route.  All against the oracle."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
import paper_2206_15014_amd as nm
from paper_2206_15014_amd import binding

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def patience(turns):
    old = binding.raw().nm_test_project_patience(turns)
    try:
        yield
    finally:
        binding.raw().nm_test_project_patience(old)


def make(rows, cols, seed, with_u=True):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((rows, cols)) * rng.random((rows, 1)) * 0.05).astype(np.float32)
    W[rng.integers(0, rows)] = 0.0
    W[:, :8] = np.round(W[:, :8] * 64) / 64                            # ties
    U = (rng.standard_normal((rows, cols)) * 0.004).astype(np.float32) if with_u else None
    return W, U


def check(got, want):
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy().view(np.uint32), w.view(np.uint32))


def padded(a, pad):
    if a is None:
        return None
    t = torch.full((a.shape[0], a.shape[1] + pad), 9.0, device="cuda")
    t[:, :a.shape[1]] = torch.from_numpy(a).cuda()
    return t[:, :a.shape[1]]


# one part (a group within one workgroup of 256 or 1024 threads, exactly full, one piece more), several parts on either, the last ones
# short or empty, a shorter last group, one group only, a width that is no power of two
SHAPES = [(70, 24, 3), (64, 256, 16), (65, 256, 17), (33, 520, 32), (300, 4096, 4), (2080, 256, 16), (800, 768, 32), (96, 3072, 32), (50, 1248, 50),
          (1000, 776, 7), (2304, 1032, 16), (4160, 520, 32), (768, 2056, 64)]


@pytest.mark.parametrize("rows, cols, rps", SHAPES)
@pytest.mark.parametrize("N, M, bits", [(2, 4, 8), (1, 4, 4), (4, 4, 8), (3, 8, 8), (2, 8, 4)])
def test_parts(rows, cols, rps, N, M, bits):
    W, U = make(rows, cols, [rows, N, M], with_u=N != 1)
    want = oracle.admm_project(W, U, N, M, bits, rps)
    Wd, Ud = padded(W, 4), padded(U, 4)
    for turns in (4096, 0):                    # meeting, and every workgroup that is early on its own
        with patience(turns):
            check(nm.nm_project(Wd, Ud, N, M, bits, rps), want)
    if U is not None:                          # in place
        Z, _, s = nm.nm_project(Wd, Ud, N, M, bits, rps, Z=torch.empty_strided(Wd.shape, Wd.stride(), device="cuda"), U_out=Ud)
        check((Z, Ud, s), want)


def test_replays_of_a_captured_call():
    W, U = make(768, 768, 1)
    Wd, Ud = torch.from_numpy(W).cuda(), torch.from_numpy(U).cuda()
    out = nm.nm_project(Wd, Ud, 2, 4, 8, 32)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            nm.nm_project(Wd, Ud, 2, 4, 8, 32, Z=out[0], U_out=out[1], scales=out[2])
    for factor in (1.0, 4.0, 0.25):            # other maxima each time
        W2 = W * np.float32(factor)
        Wd.copy_(torch.from_numpy(W2))
        nm.nm_project(Wd * 3, Ud, 2, 4, 8, 32)                         # eager calls between the replays
        graph.replay()
        torch.cuda.synchronize()
        check(out, oracle.admm_project(W2, U, 2, 4, 8, 32))


def test_calls_on_streams_side_by_side():
    """More calls in flight than regions, on three streams, with other data each."""
    data = [make(768, 768, [7, i]) for i in range(6)]
    want = [oracle.admm_project(W, U, 2, 4, 8, 32) for W, U in data]
    dev = [(torch.from_numpy(W).cuda(), torch.from_numpy(U).cuda()) for W, U in data]
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [[torch.empty(768, 768, device="cuda"), torch.empty(768, 768, device="cuda"), torch.empty(768, device="cuda")] for _ in range(90)]
    torch.cuda.synchronize()
    for i, (Z, U_out, s) in enumerate(outs):
        with torch.cuda.stream(streams[i % 3]):
            nm.nm_project(*dev[i % 6], 2, 4, 8, 32, Z=Z, U_out=U_out, scales=s)
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        check(out, want[i % 6])
