"""Plans made from freed plans' device memory give the same results, on several
streams and threads, and the memory kept for them stays bounded."""
import threading

import pytest
import torch

import workloads
from paper_2102_08463_amd import Plan

pytestmark = pytest.mark.gpu


def _once(pts, c, modes, stream=None):
    with torch.cuda.stream(stream or torch.cuda.current_stream()):
        with Plan(1, modes, eps=1e-5) as p:
            p.setpts(*pts)
            out = p.execute(c)
        return out


def test_reused_memory():
    torch.cuda.synchronize()
    sets = []
    for i, (modes, M) in enumerate([((64, 64), 20000), ((30, 41, 22), 50000), ((900,), 7000),
                                    ((64, 64), 21000)]):
        pts = [torch.from_numpy(a).float().cuda() for a in workloads.uniform(M, len(modes), i)]
        c = torch.from_numpy(workloads.strengths(M, i)).to(torch.complex64).cuda()
        sets.append((pts, c, modes))
    want = [_once(*s) for s in sets]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.default_stream())
        for rep in range(6):
            for i in range(len(sets)):
                j = (i + k + rep) % len(sets)
                got = _once(*sets[j], stream=st)
                st.synchronize()
                if not torch.equal(torch.view_as_real(got), torch.view_as_real(want[j])):
                    bad.append((k, rep, j))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad[:5]


def test_kept_memory_is_bounded():
    pts = [torch.from_numpy(a).float().cuda() for a in workloads.uniform(100000, 2, 1)]
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for n in range(200, 2200, 100):  # sizes that do not fit each other's blocks
        with Plan(2, (n, n), 8, eps=1e-5) as p:
            p.setpts(*pts)
    torch.cuda.synchronize()
    assert free0 - torch.cuda.mem_get_info()[0] <= (1 << 30) + (256 << 20)


def test_release_memory():
    from paper_2102_08463_amd import release_memory
    with Plan(1, (1024, 1024), eps=1e-5):
        pass                                 # leaves a 2048^2 grid of 33 MB behind
    held = torch.cuda.mem_get_info()[0]
    release_memory()
    assert torch.cuda.mem_get_info()[0] >= held + (32 << 20)
    pts = [torch.from_numpy(a).float().cuda() for a in workloads.uniform(5000, 2, 3)]
    c = torch.from_numpy(workloads.strengths(5000, 3)).to(torch.complex64).cuda()
    one = _once(pts, c, (64, 64))
    release_memory()
    assert torch.equal(torch.view_as_real(one), torch.view_as_real(_once(pts, c, (64, 64))))
