"""Reduction of extents above 128 by its parts: up to 192 rows one workgroup
takes all of them to 128; above, 64 waves that wait for one another's results
take the first J - 192.  What could leave a wave waiting: values that are the
wait's own marker (it is a NaN), and callers on several threads and streams at
once, whose scalars also pass through one pinned block per thread."""
import threading

import numpy as np
import pytest
import torch

from paper_1510_06689_amd import tucker

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("j", [150, 193, 200, 300, 512])
@pytest.mark.parametrize("where", ["first", "second", "last"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_nonfinite_input_ends(j, where, value):
    x = np.random.default_rng(j).standard_normal((j, 20))
    # rows that the waves finish (the second one above 193 rows), and one left to the trailing block
    x[{"first": 0, "second": min(5, max(0, j - 193)), "last": j - 1}[where], 3] = value
    d = tucker.empty_fortran(x.shape, torch.float64, "cuda:0").copy_(torch.from_numpy(x))
    for kw in ({}, {"ranks": (3, 3)}):
        with pytest.raises(tucker.TuckerError) as err:
            tucker.sthosvd(d, 1e-4, **kw)
        assert "NONFINITE" in str(err.value)
    good = tucker.sthosvd(torch.ones_like(d), 1e-4)  # and leaves nothing behind
    assert good.ranks == (1, 1)


def test_callers_at_once():
    """Four threads, each with its stream, compress tensors of their own again and
    again; every answer is that of the same call made alone, bit for bit."""
    shapes = [(301, 40, 30), (256, 200, 12), (64, 210, 20), (100, 33, 400)]
    xs, alone = [], []
    for i, s in enumerate(shapes):
        g = torch.Generator(device="cuda:0")
        g.manual_seed(i)
        core = torch.randn(5, 4, 3, generator=g, dtype=torch.float64, device="cuda:0")
        x = torch.randn(tuple(reversed(s)), generator=g, dtype=torch.float64, device="cuda:0") * 1e-3
        us = [torch.linalg.qr(torch.randn(n, r, generator=g, dtype=torch.float64, device="cuda:0"))[0]
              for n, r in zip(reversed(s), core.shape)]
        x += torch.tensordot(us[0], torch.tensordot(us[1], torch.tensordot(us[2], core, ([1], [2])), ([1], [2])), ([1], [2]))
        xs.append(x.permute(2, 1, 0))
        alone.append(tucker.sthosvd(xs[-1], 0.1))
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for n in range(12):
                    t = tucker.sthosvd(xs[i], 0.1)
                    torch.cuda.current_stream().synchronize()
                    same = (t.ranks == alone[i].ranks and t.norm2 == alone[i].norm2 and
                            list(t.discarded) == list(alone[i].discarded) and torch.equal(t.core, alone[i].core) and
                            all(torch.equal(a, b) for a, b in zip(t.factors, alone[i].factors)))
                    if not same:
                        wrong.append((i, n, t.ranks))
        except Exception as e:  # noqa: BLE001
            wrong.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(shapes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
