"""map_prune on inputs that start off a 16-byte boundary, held to the bars of
the fused-prune tests."""
import pytest
import torch

from workloads import PredictorShape, get_config, make_inputs

from gpu_util import announce, dev_inputs, device
from test_gpu_prune import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("moved", ["V", "T"])
@pytest.mark.parametrize("K", [64, 160])  # a budget that takes the candidate subset when V is aligned, and one that does not
def test_prune_inputs_off_alignment(moved, K):
    from paper_2608_06411_amd import map_prune
    cfg = get_config("sweep", B=2, N=960, M=(16, 64), K=K, K0=K // 2, pred=PredictorShape(D=512, D_h=256, d_p=64))
    announce(f"prune K={K}, {moved} off alignment")
    x = make_inputs(cfg)
    dev = device()
    d = dev_inputs(x, dev)
    flat = torch.empty(d[moved].numel() + 1, dtype=d[moved].dtype, device=dev)
    flat[1:] = d[moved].reshape(-1)
    d[moved] = flat[1:].view(d[moved].shape)  # two bytes further
    o = map_prune(d["w"], d["V"], d["pos_v"], d["T"], d["pos_t"], x["t_off"], K, K // 2, cfg.tau)
    out = {k: v.cpu() for k, v in o.items()}
    out["V_store_out"] = out["V_out"].view(torch.int16).numpy().view("uint16")
    _check(x, out, K, K // 2, cfg.tau, 2e-2)
