"""Host threads that launch on one stream at the same time, each on its own
default workspace."""

import threading

import pytest

from gpu_util import need_gpu, torch
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu


def test_threads_on_one_stream():
    dev = need_gpu()
    n = (1 << 23) + 1                                # the scan's one-pass form: a clear and a pass
    h = hm.compile("x[i]", "float: const float *x", name="wsthreads")
    hl = hm.compile("k[i]", "long: const int *k", name="wsthreads")
    stream = torch.cuda.current_stream()
    errors = []

    def work(seed):
        try:
            torch.cuda.set_device(dev)
            g = torch.Generator(device=dev)
            g.manual_seed(seed)
            with torch.cuda.stream(stream):
                k = torch.randint(-9, 9, (n,), dtype=torch.int32, device=dev, generator=g)
                x = k.float() * (2.0 ** 50 if seed % 2 else 1.0)     # second pass of the norm, or not
                sums = torch.cumsum(k, 0)
                want = torch.linalg.vector_norm(k.double()).item() * (2.0 ** 50 if seed % 2 else 1.0)
                out = torch.zeros(n, dtype=torch.int64, device=dev)
                for _ in range(30):
                    out.zero_()
                    hm.scan(hl, "a+b", "0", n, [k], out, stream=stream)
                    norm = hm.norm2(h, n, [x], stream=stream)
                    ok = torch.equal(out, sums)
                    if not ok or abs(norm.item() / want - 1) > 1e-6:
                        errors.append((seed, ok, norm.item(), want))
        except Exception as e:                       # noqa: BLE001 - reported by the main thread
            errors.append((seed, repr(e)))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not errors, errors[:3]
