"""csipm_solve_small_batch where its transforms can go wrong: prime extents
(stages of direct sums, on each axis, alone and beside other radices),
extents 1 and 2, an odd count of rows, the largest spectra that stay in LDS
and the smallest that do not, extent 64, several tiles with a ragged last one,
against the oracle's interior-point solve; and a grid outside LDS in a batch
against alone, bit for bit."""
import numpy as np
import pytest

from oracle import ipm
from paper_2502_04217_amd import workload as wl
from tests._gpu_common import need_gpu, rel2, say

pytestmark = pytest.mark.gpu

TOL = 1e-10


def _workload(shape, seed):
    rng = np.random.default_rng(seed)
    if min(shape[0] * shape[1], shape[2]) >= 3:
        return wl.make_workload(shape, n_freq=8, amplitude="normal", snr_db=20.0, half_width=-1, period=1,
                                dropout=0.15, seed=seed)
    obs = (rng.random(shape) > 0.15).astype(np.uint8)
    obs.ravel()[0] = 1
    sig = rng.standard_normal(shape) * obs
    return wl.Workload(shape, sig, obs, sig, np.zeros((0, 3), np.int64), np.zeros(0, np.complex128), 0.0)


@pytest.mark.parametrize("shape", [(11, 4, 6), (4, 13, 5), (5, 3, 11), (3, 22, 26), (1, 1, 37), (7, 1, 1), (5, 2, 2),
                                   (1, 6, 1), (3, 5, 4), (8, 8, 8), (1, 1, 1), (16, 8, 8), (3, 7, 20), (64, 2, 9), (2, 64, 3), (3, 3, 64), (27, 27, 24),
                                   (24, 24, 31), (20, 30, 32), (59, 12, 30)], ids=lambda s: "x".join(map(str, s)))
def test_shapes_match_oracle(shape):
    torch = need_gpu()
    from paper_2502_04217_amd import csipm
    w = _workload(shape, 3)
    lam = ipm.lambda_rule(w.signal, w.observed)
    beta, info = csipm.solve_small_batch(w.signal[None], w.observed[None], lambdas=[lam], tol=TOL)
    ref = ipm.ipm_solve(w.signal, w.observed, lam, ipm.IPMOptions(tol=TOL))
    err = rel2(beta[0].cpu().numpy(), ref.state.beta)
    say("small", shape, "status", info[0, 0], "ipm", info[0, 1], ref.iters, "err", err)
    assert info[0, 0] == 0 and abs(info[0, 1] - ref.iters) <= 1
    assert err <= 1e-6   # both within tol of the limit: ten times the bar of the 1e-11 solves


@pytest.mark.parametrize("shape,counts", [((30, 28, 33), (5, 40, 100, 130)), ((64, 64, 32), (2, 20))],
                         ids=["8 parts", "16 parts"])
def test_tiled_batch_bit_identical_to_one_at_a_time(shape, counts):
    """The workgroups that share a problem depend on the batch (on 256 compute
    units 8, 4, 2 and 1 of them at the first grid's counts, 16 and 8 at the
    second's): the bits do not."""
    torch = need_gpu()
    from paper_2502_04217_amd import csipm
    ws = [_workload(shape, s) for s in range(min(5, max(counts)))]
    sig, obs = (torch.tensor(np.stack(a), device="cuda") for a in ([w.signal for w in ws], [w.observed for w in ws]))
    alone = [csipm.solve_small_batch(sig[k:k + 1], obs[k:k + 1], tol=1e-8) for k in range(len(ws))]
    assert all(i[0, 0] == 0 for _, i in alone)
    for count in counts:
        say("small", shape, "count", count)
        idx = torch.arange(count, device="cuda") % len(ws)
        beta, info = csipm.solve_small_batch(sig[idx], obs[idx], tol=1e-8)
        for k in range(count):
            b1, i1 = alone[k % len(ws)]
            assert torch.equal(b1[0], beta[k]) and np.array_equal(i1[0], info[k])


def test_team_that_gives_up_is_solved_by_one_workgroup():
    """With no patience at a team's barrier every team gives up (and its count
    in the workspace says so); the results are those of patient teams."""
    torch = need_gpu()
    import ctypes as C
    from paper_2502_04217_amd import csipm
    shape, count = (30, 28, 33), 5
    ws = [_workload(shape, s) for s in range(count)]
    sig = torch.tensor(np.stack([w.signal for w in ws]), device="cuda")
    obs = torch.tensor(np.stack([w.observed for w in ws]).astype(np.uint8), device="cuda")
    want, winfo = csipm.solve_small_batch(sig, obs, lambda_frac=0.05, tol=1e-8)
    nb = csipm.small_workspace_bytes(shape, count)
    buf = torch.empty(nb // 8 + 64, dtype=torch.float64, device="cuda")
    beta = torch.empty_like(sig)
    info = torch.empty((count, csipm.SMALL_INFO), dtype=torch.float64, device="cuda")
    fn = csipm.lib().csipm_solve_small_batch_wait
    fn.restype, fn.argtypes = C.c_int, csipm.lib().csipm_solve_small_batch.argtypes + [C.c_longlong]
    off = -buf.data_ptr() % 256
    st = fn(*shape, count, sig.data_ptr(), obs.data_ptr(), None, 0.05, C.byref(csipm.default_options(tol=1e-8)),
            beta.data_ptr(), info.data_ptr(), buf.data_ptr() + off, nb, torch.cuda.current_stream().cuda_stream, -1)
    torch.cuda.synchronize()
    assert st == 0
    counts = buf.view(torch.int32)[off // 4 + 4 * sum(shape):][:16 * count:16]
    assert bool((counts >= 1 << 30).all())
    assert torch.equal(beta, want) and np.array_equal(info.cpu().numpy(), winfo)


def test_batches_of_several_threads_and_streams():
    """Cooperative launches queued by two threads on streams of their own give
    the bits of a call alone."""
    torch = need_gpu()
    import threading
    from paper_2502_04217_amd import csipm
    data = []
    for shape, count in (((30, 28, 33), 16), ((32, 32, 32), 24)):
        ws = [_workload(shape, s) for s in range(4)]
        idx = torch.arange(count, device="cuda") % 4
        sig, obs = (torch.tensor(np.stack(a), device="cuda")[idx] for a in ([w.signal for w in ws], [w.observed for w in ws]))
        data.append((sig, obs, csipm.solve_small_batch(sig, obs, tol=1e-8)[0]))
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for r in range(4):
                sig, obs, want = data[(k + r) % 2]
                if not torch.equal(csipm.solve_small_batch(sig, obs, tol=1e-8)[0], want):
                    wrong.append((k, r))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
