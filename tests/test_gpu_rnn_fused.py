"""GPU parity of the recurrent model whose hidden state fits a workgroup's registers (all time steps in one launch per
direction): hidden widths around the kernels' 64, 128 and 192 columns (193 takes the launch per step), several input
widths, one and two time steps, more examples than the backward pass has workgroups, every sampling rule."""
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_rnn import ctx, run_rnn  # noqa: F401


@pytest.mark.parametrize("hidden", [1, 33, 63, 65, 128, 129, 191, 192, 193])
@pytest.mark.parametrize("scheme,p", [(0, 1.0), (1, 0.3), (2, 0.25), (3, 0.25), (4, 0.25), (5, 0.25)])
def test_hidden_widths(ctx, hidden, scheme, p):  # noqa: F811
    from paper_2007_10412_amd import synth
    d = synth.rnn(seed=hidden + scheme, batch=5, T=6, d_input=1 + hidden % 2, hidden=hidden, classes=7, identity=False)
    run_rnn(ctx, d, scheme, p, seed=3)


@pytest.mark.parametrize("batch,T,d_input,hidden", [(520, 3, 1, 20), (1030, 2, 8, 70), (4, 1, 3, 150), (3, 2, 8, 180)])
def test_batches_steps_and_inputs(ctx, batch, T, d_input, hidden):  # noqa: F811
    from paper_2007_10412_amd import synth
    d = synth.rnn(seed=batch, batch=batch, T=T, d_input=d_input, hidden=hidden, classes=10, identity=False)
    run_rnn(ctx, d, 3, 0.3, seed=4, check_store=T > 1)
