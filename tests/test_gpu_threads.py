"""Checks of one context from several host threads: each gets its own answer."""
import threading

import numpy as np
import pytest

import tc_inputs
from gpu_common import make_pair, to_dev

pytestmark = pytest.mark.gpu


def test_finite_checks_from_several_threads():
    S, P, cfg = make_pair("small")
    u = tc_inputs.initial_state(P.r, cfg)
    S.set_state(to_dev(u))
    good = S.diag()
    u[2, 3, 1, 1] = complex(np.nan, 0.0)
    S.set_state(to_dev(u))
    finite, cfl = [], []

    def check():
        for _ in range(200):
            finite.append(S.check_finite())

    def diag():
        for _ in range(200):
            cfl.append(S.diag()["slip"])

    threads = [threading.Thread(target=f) for f in (check, check, check, diag)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    S.close()
    print(f"{sum(finite)} of {len(finite)} checks missed the value")
    assert len(finite) == 600 and not any(finite)
    assert cfl == [good["slip"]] * 200
