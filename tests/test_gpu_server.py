"""Continuous-batching server: jobs that arrive while others are on the GPU
join the next tile round; every job's result must equal the oracle and the
same job run alone (tolerance 0), admission must back off when the arena is
full and refuse jobs that can never fit."""
import numpy as np
import pytest

import oracle
from paper_1311_0378_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import DEV, first_mismatch  # noqa: E402
from paper_1311_0378_amd import mrecon  # noqa: E402
from test_gpu_batch import make_batch, oracle_of  # noqa: E402


def alone(job, conn):
    kind, a, m = job
    d = torch.from_numpy(a).to(DEV)
    if kind == "recon":
        mrecon.recon_dilate(d, torch.from_numpy(m).to(DEV), conn)
    else:
        mrecon.fill_holes(d, conn)
    return d.cpu().numpy()


def run_server(jobs, arena, conn=8, per_step=3, dtype=torch.uint8, max_jobs=16, rounds=None):
    srv = mrecon.Server(arena, max_jobs=max_jobs, dtype=dtype, conn=conn, rounds_per_step=rounds)
    pending = list(enumerate(jobs))
    ids, results, eagain = {}, {}, 0
    steps = 0
    while pending or srv.stats()["resident"]:
        # a few arrivals per step, so new jobs join rounds already running
        for _ in range(per_step):
            if not pending:
                break
            i, (kind, a, m) = pending[0]
            jid = srv.submit(a, m if kind == "recon" else None)
            if jid is None:
                eagain += 1
                break
            ids[jid] = i
            pending.pop(0)
        srv.step()
        steps += 1
        for jid, res in srv.poll():
            results[ids[jid]] = res.numpy()
        assert steps < 100000
    srv.close()
    return results, eagain


@pytest.mark.parametrize("rounds", [1, 2, 3, None], ids=lambda r: f"rounds{r}")
@pytest.mark.parametrize("conn", [4, 8])
def test_server_results_equal_alone_and_oracle(conn, rounds):
    jobs = make_batch(30, "u8", seed=11 + conn, lo=20, hi=600)
    print(f"[gpu] server 30 jobs conn{conn} rounds/step {rounds}", flush=True)
    results, _ = run_server(jobs, 256 << 20, conn=conn, rounds=rounds)
    assert len(results) == len(jobs)
    for i, job in enumerate(jobs):
        want = oracle_of(job, conn)
        assert np.array_equal(results[i], want), f"job {i}: " + first_mismatch(results[i], want)
        assert np.array_equal(results[i], alone(job, conn)), f"job {i} differs from its solo run"


def test_server_i32():
    jobs = make_batch(12, "i32", seed=4, lo=20, hi=300)
    results, _ = run_server(jobs, 128 << 20, dtype=torch.int32)
    for i, job in enumerate(jobs):
        assert np.array_equal(results[i], oracle_of(job, 8)), f"job {i}"


def test_server_backpressure_and_reject():
    # 16 jobs of about 7 MiB in all through a 3 MiB arena
    jobs = make_batch(16, "u8", seed=2, lo=200, hi=900)
    results, eagain = run_server(jobs, 3 << 20, per_step=16)
    assert eagain > 0, "a small arena must push back"
    assert len(results) == len(jobs)
    for i, job in enumerate(jobs):
        assert np.array_equal(results[i], oracle_of(job, 8)), f"job {i}"
    srv = mrecon.Server(8 << 20, max_jobs=4)
    big = np.zeros((4000, 4000), np.uint8)
    with pytest.raises(mrecon.MrError) as e:
        srv.submit(big, big)
    assert e.value.code == mrecon.MR_EINVAL
    srv.close()


def test_server_windows_of_a_larger_image():
    # jobs given as windows of one pinned image (host row pitch > width),
    # results written into windows of one pinned output
    big_m, big_k = synth.make_tile(700, 900, 60, 5, "u8", 0.0)
    big_f = synth.binary_from_mask(synth.quantize(synth.make_field(700, 900, 60, 6, 0.3), "u8"))
    tm, tk, tf = (torch.from_numpy(x).pin_memory() for x in (big_m, big_k, big_f))
    out = torch.zeros((700, 900), dtype=torch.uint8, pin_memory=True)
    outf = torch.zeros((700, 900), dtype=torch.uint8, pin_memory=True)
    wins = [(0, 0, 300, 400), (310, 17, 390, 233), (50, 500, 129, 400), (400, 300, 300, 600)]
    srv = mrecon.Server(64 << 20, max_jobs=8)
    ids = {}
    for k, (y, x, h, w) in enumerate(wins):
        sl = (slice(y, y + h), slice(x, x + w))
        ids[srv.submit(tm[sl], tk[sl], out=out[sl])] = ("recon", sl)
        ids[srv.submit(tf[sl], out=outf[sl])] = ("fill", sl)
        if k == 1:
            srv.step()
    srv.drain()
    got = dict(srv.poll())
    srv.close()
    assert sorted(got) == sorted(ids)
    for jid, (kind, sl) in ids.items():
        if kind == "recon":
            want = oracle.recon_dilate(np.ascontiguousarray(big_m[sl]),
                                       np.ascontiguousarray(big_k[sl]), 8)[0]
            src = out
        else:
            want = oracle.fill_holes(np.ascontiguousarray(big_f[sl]), 8)[0]
            src = outf
        assert np.array_equal(src[sl].numpy(), want), f"{kind} window {sl}"
        # pixels outside the windows were never written
    mask = np.zeros((700, 900), bool)
    for _, (_, sl) in ids.items():
        mask[sl] = True
    assert not out.numpy()[~mask].any() and not outf.numpy()[~mask].any()


# More device jobs than one admission launch takes, all in one step: windows of one
# plane at any byte alignment, read where they are, with the results over the inputs.
def test_server_device_jobs_in_place():
    jobs = make_batch(35, seed=71, lo=1, hi=300)
    big = torch.full((2, 400, 35 * 301), 5, dtype=torch.uint8, device=DEV)
    srv = mrecon.Server(256 << 20, max_jobs=40)
    wins, ids = [], {}
    for i, (kind, a, m) in enumerate(jobs):
        win = (slice(i, i + a.shape[0]), slice(301 * i, 301 * i + a.shape[1]))
        big[0][win] = torch.from_numpy(a).to(DEV)
        if m is not None:
            big[1][win] = torch.from_numpy(m).to(DEV)
        wins.append(win)
    torch.cuda.synchronize()
    for i, (kind, a, m) in enumerate(jobs):
        d, k = big[0][wins[i]], big[1][wins[i]] if m is not None else None
        ids[srv.submit(d, k, out=d)] = i
    assert None not in ids and len(ids) == len(jobs)
    print("[gpu] server device jobs in place", flush=True)
    srv.drain()
    got = {ids[j]: res for j, res in srv.poll()}
    for i, job in enumerate(jobs):
        want = oracle_of(job, 8)
        res = got[i].cpu().numpy()
        assert np.array_equal(res, want), f"job {i}: " + first_mismatch(res, want)
        got[i].fill_(5)
    srv.close()
    assert bool((big[0] == 5).all())


# A result that is an input of another job in flight: both see what the buffer held when
# they were submitted, whichever comes first and whether or not its rounds have begun.
@pytest.mark.parametrize("steps", [0, 1])
@pytest.mark.parametrize("reader_first", [False, True])
def test_server_device_jobs_share_buffers(reader_first, steps):
    from test_oracle_pins import serpentine
    marker, mask = serpentine(500, 700, 8)  # a long chain: the reader ends last
    x = torch.from_numpy(mask).to(DEV)
    writer = (x, None, mrecon.MR_OP_FILL, x)
    reader = (torch.from_numpy(marker).to(DEV), x, mrecon.MR_OP_RECON,
              torch.zeros_like(x))
    srv = mrecon.Server(64 << 20, max_jobs=4)
    torch.cuda.synchronize()
    print(f"[gpu] shared buffers reader_first={reader_first} steps={steps}", flush=True)
    if reader_first:
        srv.submit(*reader[:3], out=reader[3])
        for _ in range(steps):
            srv.step()
        srv.submit(*writer[:3], out=writer[3])
    else:
        srv.submit(*writer[:3], out=writer[3])
        srv.submit(*reader[:3], out=reader[3])
    srv.drain()
    srv.close()
    want = oracle.recon_dilate(marker, mask, 8)[0]
    assert np.array_equal(reader[3].cpu().numpy(), want), first_mismatch(reader[3].cpu().numpy(),
                                                                         want)
    want = oracle.fill_holes(mask, 8)[0]
    assert np.array_equal(x.cpu().numpy(), want), first_mismatch(x.cpu().numpy(), want)


def queue_upload(srv, side=8192):
    """A job that keeps the server's input copies busy for a millisecond or more."""
    z = torch.zeros((side, side), dtype=torch.uint8, pin_memory=True)
    return z, srv.submit(z, z)


# Device jobs' inputs overwritten before their rounds have begun, by work on the server's
# stream or after a wait for the device: each job still sees what it was submitted with.
@pytest.mark.parametrize("wait", [False, True])
def test_server_device_inputs_overwritten_after_submit(wait):
    jobs = make_batch(8, seed=5, lo=60, hi=700)
    want = [oracle_of(j, 8) for j in jobs]
    dev = [(torch.from_numpy(a).to(DEV), torch.from_numpy(m).to(DEV) if m is not None else None)
           for _, a, m in jobs]
    srv = mrecon.Server(512 << 20, max_jobs=16)
    torch.cuda.synchronize()
    print(f"[gpu] server inputs overwritten wait={wait}", flush=True)
    keep, big = queue_upload(srv)
    ids = {srv.submit(a, m): i for i, (a, m) in enumerate(dev)}
    if wait:
        torch.cuda.synchronize()
    for a, m in dev:
        a.fill_(255)
        if m is not None:
            m.fill_(255)
    srv.drain()
    got = dict(srv.poll())
    srv.close()
    assert not got.pop(big).any() and sorted(got) == sorted(ids)
    for jid, i in ids.items():
        res = got[jid].cpu().numpy()
        assert np.array_equal(res, want[i]), f"job {i}: " + first_mismatch(res, want[i])


def ring(side):
    """An image whose hole is all of its inside."""
    a = np.full((side, side), 255, np.uint8)
    a[1:-1, 1:-1] = 0
    return a


# A reader of the buffer that a job submitted before it fills: the writer's rounds are done,
# its result is not written yet, and the reader's input copies wait behind an upload.
@pytest.mark.parametrize("steps", [0, 1])
def test_server_result_waits_for_its_readers(steps):
    x = torch.from_numpy(ring(300)).to(DEV)
    marker = torch.full_like(x, 77)
    out = torch.zeros_like(x)
    srv = mrecon.Server(512 << 20, max_jobs=4)
    torch.cuda.synchronize()
    print(f"[gpu] result waits for its readers steps={steps}", flush=True)
    srv.submit(x, None, mrecon.MR_OP_FILL, out=x)
    for _ in range(steps):
        srv.step()
    torch.cuda.synchronize()
    keep, _ = queue_upload(srv)
    srv.submit(marker, x, mrecon.MR_OP_RECON, out=out)
    srv.drain()
    srv.close()
    want = np.minimum(ring(300), 77)
    assert np.array_equal(out.cpu().numpy(), want), first_mismatch(out.cpu().numpy(), want)
    assert bool((x == 255).all())


# A reader of a buffer that a finished job's result is on its way to, behind a larger
# result: it sees the whole result.
def test_server_reader_waits_for_a_result_under_way():
    full = torch.full((8192, 8192), 255, dtype=torch.uint8, pin_memory=True)
    x = torch.zeros((300, 300), dtype=torch.uint8, pin_memory=True)
    srv = mrecon.Server(512 << 20, max_jobs=4)
    print("[gpu] reader waits for a result under way", flush=True)
    srv.submit(full)
    srv.submit(torch.from_numpy(ring(300)).pin_memory(), out=x)
    srv.step()
    torch.cuda.synchronize()
    srv.step()  # both results are enqueued, the larger one first
    j = srv.submit(x)
    srv.drain()
    res = dict(srv.poll())[j].numpy()
    srv.close()
    assert (x.numpy() == 255).all()
    assert (res == 255).all(), first_mismatch(res, np.full_like(res, 255))


@pytest.mark.parametrize("conn", [4, 8])
def test_server_device_jobs(conn):
    # jobs whose inputs and results are device memory (MR_JOB_DEVICE): the
    # same answers as the oracle; inputs are windows with a row pitch wider
    # than the job, results land in pitched device buffers
    jobs = make_batch(24, seed=40 + conn)
    want = [oracle_of(j, conn) for j in jobs]
    srv = mrecon.Server(256 << 20, max_jobs=8, conn=conn)
    pending = list(range(len(jobs)))
    owned, got = {}, {}
    keep = []
    print(f"[gpu] server device jobs conn{conn}", flush=True)
    while pending or owned:
        while pending:
            i = pending[0]
            kind, a, m = jobs[i]
            H, W = a.shape
            big = torch.zeros((H, W + 37), dtype=torch.uint8, device=DEV)
            big[:, :W] = torch.from_numpy(a).to(DEV)
            d = big[:, :W]
            mk = None
            if kind == "recon":
                bigm = torch.zeros_like(big)
                bigm[:, :W] = torch.from_numpy(m).to(DEV)
                mk = bigm[:, :W]
            out = torch.full((H, W + 5), 7, dtype=torch.uint8, device=DEV)[:, :W]
            jid = srv.submit(d, mk, out=out)
            if jid is None:
                break
            keep.append((big, mk, out))
            owned[jid] = i
            pending.pop(0)
        srv.step()
        for jid, res in srv.poll():
            got[owned.pop(jid)] = res.cpu().numpy()
    srv.close()
    for i in range(len(jobs)):
        assert np.array_equal(got[i], want[i]), f"job {i}: " + first_mismatch(got[i], want[i])
