"""GPU parity of the register-held recurrent model where two workgroups share a compute unit (more examples than units,
hidden 65 to 128: rows of the state padded to 144), on both sides of the line and at one and more time steps, with the
waves off the chain ahead of (T = 1, 2), at (3, 4) and behind their prefetch distance.  Tolerances are run_rnn's."""
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_rnn import ctx, run_rnn  # noqa: F401


@pytest.mark.parametrize("batch", [256, 257])
@pytest.mark.parametrize("hidden", [65, 100, 128])
@pytest.mark.parametrize("T,d_input,scheme,p", [(1, 1, 3, 0.3), (2, 1, 5, 0.25), (3, 3, 1, 0.3), (4, 1, 0, 1.0), (9, 1, 2, 0.25)])
def test_two_workgroups_a_unit(ctx, batch, hidden, T, d_input, scheme, p):  # noqa: F811
    from paper_2007_10412_amd import synth
    d = synth.rnn(seed=batch + hidden + T, batch=batch, T=T, d_input=d_input, hidden=hidden, classes=7, identity=False)
    run_rnn(ctx, d, scheme, p, seed=6, check_store=T > 1)
