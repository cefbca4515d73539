"""Two host threads on two streams at once: solves and coding calls share the library's
pool of device memory and its list of pinned blocks, so memory freed on one stream is
used on the other and a block goes from thread to thread.  Every result equals the one of the same
call by itself."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_18147_amd import ecasq, inputs

pytestmark = pytest.mark.gpu

INFO = ("t", "p", "lambda", "mse", "entropy", "dp_solves", "status")


def _result(r):
    """A call's outputs on the host, in a form that == compares."""
    out = []
    for v in r:
        if isinstance(v, torch.Tensor):
            out.append(v.cpu().numpy().tobytes())
        elif isinstance(v, dict):
            out.append(tuple(v[k] for k in INFO))
        else:
            out.append(v)
    return out


def _jobs():
    dev = "cuda"
    small = torch.from_numpy(inputs.normal(1024, 1)).to(dev)
    mid = torch.from_numpy(inputs.lognormal_signed(6000, 2)).to(dev)
    wide = torch.from_numpy(inputs.normal(20000, 3)).to(dev)
    half = torch.from_numpy(inputs.normal(30000, 4)).to(dev).to(torch.bfloat16)
    sym = torch.from_numpy(np.random.default_rng(5).integers(0, 9, 50000).astype(np.uint8)).to(dev)
    cb = torch.linspace(-3, 3, 17, dtype=torch.float64, device=dev)
    grid = ecasq.ecasq_default_options(alphabet=2, alphabet_size=2000)

    def code():
        s = ecasq.ecasq_encode(sym, 9)
        return s, ecasq.ecasq_decode(s, sym.numel(), 9)

    return [
        ("solve 1024", lambda: ecasq.ecasq_solve(small, 16, 2.0)),
        ("solve 6000", lambda: ecasq.ecasq_solve(mid, 12, 1.5)),
        ("grid 20000", lambda: ecasq.ecasq_solve(wide, 24, 2.5, options=grid)),
        ("fixed 30000 bf16", lambda: ecasq.ecasq_solve_lagrangian(half, 32, 0.1)),
        ("optimal 1024", lambda: ecasq.ecasq_solve_optimal(small, 8, 0.05)),
        ("round 50000", lambda: ecasq.ecasq_quantize(wide.repeat(3)[:50000], cb, 7)),
        ("code 50000", code),
    ]


def test_two_threads_two_streams():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jobs = _jobs()
    want = {}
    for name, job in jobs:
        print("[case] alone", name, flush=True)
        want[name] = _result(job())
    torch.cuda.synchronize()
    wrong, stop = [], threading.Event()

    def work(order):
        st = torch.cuda.Stream()
        try:
            with torch.cuda.stream(st):
                for name, job in order:
                    if stop.is_set():
                        return
                    got = _result(job())
                    st.synchronize()
                    if got != want[name]:
                        raise AssertionError(f"{name} differs")
        except BaseException as e:  # reported by the main thread
            wrong.append(e)
            stop.set()

    print("[case] two threads", flush=True)
    ts = [threading.Thread(target=work, args=((jobs * 6)[k:] + jobs[:k],)) for k in (0, 3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in ts)
    assert not wrong, wrong[0]


def test_trim_gives_memory_back():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(inputs.normal(1 << 18, 6)).to("cuda").to(torch.bfloat16)
    cb = ecasq.ecasq_solve_optimal(x, 16, 0.1)[0]  # hundreds of MB of tables
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ecasq.ecasq_trim()
    after = torch.cuda.mem_get_info()[0]
    print("[case] trim", before, after, flush=True)
    assert after > before
    ecasq.ecasq_trim()  # nothing kept
    assert torch.equal(ecasq.ecasq_solve_optimal(x, 16, 0.1)[0], cb)
