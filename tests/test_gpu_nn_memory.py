"""The second activation set of Gram-form training (kept where memory allows): the gradient does not
depend on it, it is no reason for a call to fail, and it does not stay after training."""
import numpy as np
import pytest

import synth
from gpu_helpers import DEV

torch = pytest.importorskip("torch")
from paper_1409_1510_amd import hisq  # noqa: E402

pytestmark = pytest.mark.gpu

DIMS, N, L = (8, 8, 8, 8), 8, 2
VH = int(np.prod(DIMS)) // 2
ACT = N * 3 * 2 * VH * 16 * 2        # one BF16 activation
LINKS = 2 * VH * 144 * (8 + 4)       # FP32 and FP16 copies, both parities
SCRATCH = 11 * N * 3 * VH * 8 + (1024 + 1) * 256 * 8  # vectors and partial sums of a gradient
MANDATORY = LINKS + SCRATCH + (2 * L + 2) * ACT
TUNE = 2 * N * 3 * VH * 8            # vectors of the launch tuner (residual loss, first call)
SLACK = 1 << 18                      # weights, partials, rounding of the sizes above


def _network(loss):
    fat, naik = synth.gauge_links(DIMS, 92)
    lat = hisq.Lattice(DIMS, 0)
    lat.load_links(fat, naik, hisq.HISQ_LINKS_F32 | hisq.HISQ_LINKS_F16)
    lib = hisq.library()
    hisq._check(lat.ctx, lib.hisq_nn_init(lat.ctx, L, 8, 7))
    hisq._check(lat.ctx, lib.hisq_nn_set_form(lat.ctx, hisq.HISQ_NN_FORM_GRAM))
    hisq._check(lat.ctx, lib.hisq_nn_set_loss(lat.ctx, loss, 0.3))
    return lat


def _pairs():
    return [torch.from_numpy(synth.sources(DIMS, N, s)).to(DEV) for s in (5, 6)]


def _loss_grad(lat, r, y):
    lib = hisq.library()
    loss, grad = hisq.ctypes.c_double(), (hisq.ctypes.c_double * (2 * lib.hisq_nn_num_params(lat.ctx)))()
    hisq.hisq_set_stream(lat.ctx)
    hisq._check(lat.ctx, lib.hisq_nn_loss_grad(lat.ctx, N, hisq._ptr(r), hisq._ptr(y),
                                               hisq.ctypes.byref(loss), grad))
    return loss.value, np.array(grad[:])


@pytest.mark.parametrize("loss", [hisq.HISQ_NN_LOSS_SOLUTION, hisq.HISQ_NN_LOSS_RESIDUAL])
def test_gradient_is_the_same_with_and_without_the_second_set(loss):
    """No limit (second set kept), a limit that leaves no room for it (the forward pass again), and one
    that holds it but not the launch tuner's vectors beside it (given back in the middle of the
    first call where the loss applies M): same bits, no error text, and the call that follows too."""
    r, y = _pairs()
    assert TUNE > 2 * SLACK
    ref = None
    for limit in (0, MANDATORY + TUNE + SLACK, MANDATORY + 2 * L * ACT + SLACK):
        lat = _network(loss)
        hisq.hisq_set_memory_limit(lat.ctx, limit)
        for _ in range(2):
            got = _loss_grad(lat, r, y)
            ref = ref or got
            assert got[0] == ref[0] and np.array_equal(got[1], ref[1]), limit
        assert hisq.hisq_last_error(lat.ctx) == ""
        lat.close()


def test_limit_below_the_mandatory_buffers_is_refused():
    r, y = _pairs()
    lat = _network(hisq.HISQ_NN_LOSS_SOLUTION)
    hisq.hisq_set_memory_limit(lat.ctx, LINKS + SLACK)
    with pytest.raises(hisq.HisqError) as e:
        _loss_grad(lat, r, y)
    assert e.value.code == hisq.HISQ_ERR_OOM
    hisq.hisq_set_memory_limit(lat.ctx, 0)
    _loss_grad(lat, r, y)
    lat.close()


def test_training_gives_the_second_set_back():
    """At 16^4 with 8 pairs a second set of 4 layers takes 402 MB: device memory before and after a
    training call differ by what training needs without it."""
    dims, n, layers = (16, 16, 16, 16), 8, 4
    vh = int(np.prod(dims)) // 2
    act = n * 3 * 2 * vh * 16 * 2
    lat = hisq.Lattice(dims, 0)
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    links = 0.3 * torch.randn(2 * vh, 4, 3, 3, generator=g, dtype=torch.complex128, device=DEV)
    lat.load_links(links, links, hisq.HISQ_LINKS_F32 | hisq.HISQ_LINKS_F16)
    lib = hisq.library()
    hisq._check(lat.ctx, lib.hisq_nn_init(lat.ctx, layers, 8, 7))
    hisq._check(lat.ctx, lib.hisq_nn_set_form(lat.ctx, hisq.HISQ_NN_FORM_GRAM))
    r = torch.randn(n, 3, vh, generator=g, dtype=torch.complex128, device=DEV)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    hisq.hisq_set_stream(lat.ctx)
    hisq._check(lat.ctx, lib.hisq_nn_train(lat.ctx, n, hisq._ptr(r), hisq._ptr(r), 1, n, 1e-3, 1, None))
    torch.cuda.synchronize()
    held = free0 - torch.cuda.mem_get_info()[0]
    need = (2 * layers + 2) * act + 11 * n * 3 * vh * 8
    assert held <= need + (64 << 20), (held, need)
    lat.close()
