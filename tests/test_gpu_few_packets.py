"""Runs that do not fill the chip, whose wavefronts hold fewer packets than
lanes: packet counts around one per wavefront and around a full chip, every
packet traced against the oracle (bars as in test_gpu_parity.py), spheres
(ids reserved in chunks) and aligned grains (ids as needed), with the default
schedule and with explicit block sizes and scattering batches."""
import pytest

from parity_util import compare_traces, gpu_run, say
from test_gpu_tally_layout import odd_box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle as o
    o.lib()
    return o


@pytest.mark.parametrize("grains,tol", [("sphere", 1e-12), ("aligned", 1e-10)])
@pytest.mark.parametrize("packets,opts", [(1, {}), (2, {}), (63, {}), (2049, {}), (3072, {}), (3073, {}), (6145, {}),
                                          (9000, dict(block_size=64)), (9000, dict(blocks_per_cu=1, scatter_batch=64)),
                                          (700, dict(blocks_per_cu=1, scatter_batch=1, scatter_wait=1))])
def test_paths(O, grains, tol, packets, opts):
    cfg = odd_box(packets=packets, grains=grains)
    say(f"case: {grains}, {packets} packets, {opts}")
    ctx = gpu_run(cfg, trace_packets=packets, transport_fp64=1, **opts)
    try:
        _, _, tr_o, st_o = O.run(cfg, traces=True)
        compare_traces(ctx.traces(), tr_o, tol, 1.0, f"{grains} {packets}")
        assert ctx.stats()["packets"] == packets
        assert ctx.stats()["cell_steps"] == st_o["cell_steps"]
    finally:
        ctx.close()
