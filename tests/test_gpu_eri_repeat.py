"""The dense tensor has one value per element: the same bits in every call, on
whatever stream and in every replay of a capture, and in all eight places that
permutations of the indices give it.  The molecules have d shells, whose short
(dd|dd) lists several blocks share."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_common import announce, need_gpu, torch, zeros  # noqa: E402

from mess_inputs import generators as G  # noqa: E402

pytestmark = pytest.mark.gpu

SYSTEMS = {"water1": lambda: G.water_cluster(0, n_waters=1, box=4.0),
           "water3": lambda: G.water_cluster(0, n_waters=3, box=8.0)}


def _symmetric(t):
    return all(torch.equal(t, t.permute(p)) for p in ((1, 0, 2, 3), (0, 1, 3, 2), (2, 3, 0, 1)))


@pytest.mark.parametrize("system", list(SYSTEMS))
@pytest.mark.parametrize("prec", [0, 1])
def test_tensor_repeats_and_is_symmetric(system, prec):
    mess = need_gpu()
    B = mess.basis_from_molecule(SYSTEMS[system]())
    N = B.nbf
    announce(f"eri repeat {system} prec={prec} nbf={N}")
    first = zeros(N, N, N, N)
    mess.mess_eri(B, first, prec=prec, schwarz_tol=0.0)
    assert _symmetric(first)
    # calls on two streams in turn, none waited for: the workspace of one must
    # not be taken by the next before it is read
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    outs = [zeros(N, N, N, N) for _ in range(6)]
    torch.cuda.synchronize()
    for k, out in enumerate(outs):
        with torch.cuda.stream(streams[k % 2]):
            mess.mess_eri(B, out, prec=prec, schwarz_tol=0.0)
    torch.cuda.synchronize()
    for out in outs:
        assert torch.equal(out, first)
    B.close()


def test_tensor_of_a_replay():
    mess = need_gpu()
    B = mess.basis_from_molecule(SYSTEMS["water3"]())
    N = B.nbf
    announce(f"eri replay nbf={N}")
    eager, out = zeros(N, N, N, N), zeros(N, N, N, N)
    mess.mess_eri(B, eager, schwarz_tol=0.0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mess.mess_eri(B, out, schwarz_tol=0.0)
    seen = []
    for _ in range(3):
        out.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        seen.append(out.clone())
        # work of its own between the replays
        mess.mess_eri(B, eager, schwarz_tol=0.0)
        torch.cuda.synchronize()
    assert _symmetric(seen[0])
    assert all(torch.equal(s, seen[0]) for s in seen)
    # another order of the same 1296 terms
    assert torch.max(torch.abs(seen[0] - eager)) <= 1e-12 * torch.max(torch.abs(eager))
    B.close()
