"""A schedule change between lbm_step and ibm_couple is refused and changes
nothing: the coupling still follows the stream order of its lattice step (FP16
with the full-precision box, whose step and correction would otherwise run side
by side), and a captured graph stays."""
import ctypes as C

import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("serial", [0, 1])
def test_refused_change_of_the_stream_order_leaves_the_step(serial):
    import torch
    from paper_2408_15115_amd import turret as T
    case = W.make_case(40, 36, 44, 0.7, W.BC_FREESLIP, W.BC_FREESLIP, 4, 2e-5)
    body = W.sphere_fibonacci_body(4.0, 300, 2.0, [19.5, 17.5, 22.0])
    S, ref = (T.Solver([case], [body], storage="f16", serial_ibm=serial, stream=torch.cuda.Stream()) for _ in range(2))
    S.graph_capture(2)
    for _ in range(6):
        for s in (S, ref):
            s.body_advance()
            s.lbm_step()
            if s is S:
                o = T.make_options("f16", serial_ibm=1 - serial, collision=1, fine_box=1)
                assert T.lbm_set_schedule(S._ctx, C.byref(o)) == T.LBM_ESTATE
            s.ibm_couple()
            s.window_shift()
    S.graph_launch()   # (an even number of steps: the buffers stand as at the capture)
    ref.run(2)
    a, b = S.body_state(), ref.body_state()
    assert all(np.array_equal(a[k], b[k]) for k in a)
    assert np.array_equal(S.populations(), ref.populations())
    S.close()
    ref.close()
