"""The width-128 BF16 / FP8 sampler, whose waves carry 32 samples each: a sample's result does not
depend on the launch's size (edges of a 32-sample tile, fewer tiles than CUs, several tiles to a
wave), nor on whether its noise comes from the generator or from memory, nor on the raw output
being asked for.  All comparisons are bit for bit."""
import numpy as np
import pytest
import torch

from paper_2512_13965_amd import inputs
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

N = 150_001          # beyond one tile to each of 256 * 12 waves


@pytest.mark.parametrize("integrator,K", [("euler", 3), ("rk4", 2)])
@pytest.mark.parametrize("precision,n_in", [("bf16", 10), ("fp8", 10), ("bf16", 11), ("bf16", 12)])
def test_results_do_not_depend_on_the_launch(precision, n_in, integrator, K):
    binding = require_gpu()
    m = binding.Model(inputs.pack_blob(inputs.random_weights(128, 3, n_in=n_in)), precision)
    if n_in == 12:
        cond = binding.DeviceCondInternal.from_host(inputs.internal_conditions(N, 9))
        call = binding.gmc_sample_internal
    else:
        la = (-1.0, 1.0) if n_in == 11 else None
        cond = binding.DeviceCond.from_host(inputs.transmission_conditions(N, 9, log_aspect_range=la))
        call = binding.gmc_sample
    def run(n, id_base=0, **kw):
        raw = torch.full((5, n), 7.0, device="cuda")
        r = call(m, cond, integrator, K, 4, id_base, n=n, raw=raw, **kw).to_host()
        return dict(r, raw=raw.cpu().numpy())

    want = run(N)
    assert np.isfinite(want["raw"]).all()
    for n in (1, 31, 32, 33, 257, 8191, 16_384, 16_385, 98_337):
        got = run(n)
        for k in want:
            np.testing.assert_array_equal(got[k], want[k][..., :n], err_msg=f"{k}, {n} samples")
    plain = call(m, cond, integrator, K, 4, 0).to_host()
    for k in plain:
        np.testing.assert_array_equal(plain[k], want[k], err_msg=k)
    # explicit noise: equal rows give equal results wherever they stand in the launch
    z = torch.from_numpy(inputs.noise(64, 2)).cuda()
    zz = z.repeat(1, 3).contiguous()
    sub = type(cond)(*[None if v is None else v[:64].repeat(3).contiguous() for v in vars(cond).values()])
    raw = torch.empty(5, 192, device="cuda")
    call(m, sub, integrator, K, 4, 0, noise=zz, raw=raw)
    assert torch.equal(raw[:, :64], raw[:, 64:128]) and torch.equal(raw[:, :64], raw[:, 128:])
    m.close()


@pytest.mark.parametrize("precision,split,graphs", [("bf16", True, False), ("fp8", True, True), ("bf16", False, True)])
def test_transport_does_not_depend_on_who_chooses(precision, split, graphs):
    """Counts that only the device knows (a split step's collided crossings, a captured step's
    count) choose between teams and waves there when the host's bound exceeds 64 samples per
    compute unit.  A bank of all histories takes both choices as the count falls, a bank of 64 per
    compute unit only ever runs teams; the tallies agree up to the order of their FP64 additions
    (n terms of at most 1 each)."""
    from paper_2512_13965_amd import transport
    binding = require_gpu()
    few = 64 * torch.cuda.get_device_properties(0).multi_processor_count
    prob = inputs.checkerboard_problem(16, src=2)
    n = 5 * few // 2
    m = binding.Model(inputs.pack_blob(inputs.random_weights(128, 31, flags=2 if split else 0)), precision)
    out = []
    for cap in (4 * few, few):
        w = binding.World(cap, 1, 1 << 12)
        w.set_graphs(graphs)
        out.append(transport.run_problem(w, prob, n, 5, binding.SAMPLER_GMC, m, 4, chunk=cap))
        w.close()
    m.close()
    a, b = out
    assert a["transmissions"] == b["transmissions"]
    for k in ("flux", "absorbed", "leak", "cutoff", "wpath", "path", "visits"):
        np.testing.assert_allclose(a[k], b[k], rtol=1e-12, atol=1e-12 * n, err_msg=k)
