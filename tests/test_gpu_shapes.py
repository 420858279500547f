"""GPU parity at the sizes where the kernels' dispatch changes or their tiles end: stage by stage against the oracle,
with the tolerances of test_gpu_parity (bf16 2e-2, fp32 1e-5 of the reference's maximum, also per expert and bucket)."""
import pytest

from paper_2304_03946_amd import workloads as W
from test_gpu_parity import api, run_stagewise  # noqa: F401  (api: module fixture)

pytestmark = pytest.mark.gpu


def stagewise(api, cfg, seed=3):  # noqa: F811
    inp = W.make_layer_inputs(cfg, seed=seed)
    run_stagewise(api, cfg, inp, *W.placement_from_loads(W.prior_loads(cfg, seed), cfg.V, cfg.max_rep, shuffle_seed=11))


# one job per 1/8 and 1/4 of a patch: the work lists are dealt out over 64 and 32 bins (several lanes rows of the
# minimum); two patches per job: 4 bins; 70 jobs: the second pass of 64
@pytest.mark.parametrize("N,d,f,E,V", [(2100, 256, 1024, 12, 17), (1300, 256, 2048, 6, 9), (4200, 512, 1024, 5, 8), (3000, 256, 512, 70, 80)])
def test_weight_gradient_work_lists(api, N, d, f, E, V):  # noqa: F811
    stagewise(api, W.scaled(W.CONFIGS["gpt_m"], N=N, d=d, f=f, E=E, V=V, max_rep=3))
