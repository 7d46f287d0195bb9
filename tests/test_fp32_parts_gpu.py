"""fp32 products formed from bf16 parts (head width times tile slots 2048, one slot wave): what
they must share with the fp32 matrix instruction beyond an error bound (needs an MI355X)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paritycheck import announce
from test_parity_gpu import run_gpu, small

pytestmark = pytest.mark.gpu

SHAPES = [(32, 64), (32, 48), (64, 32)]


@pytest.mark.parametrize("D,G", SHAPES)
@pytest.mark.parametrize("N", [1000, 33])
def test_passes_share_their_logits(D, G, N):
    """The slice forms a logit with the points as rows, the deslice with the slots as rows; both
    must get the same fp32 number, since every other pass recomputes weights against the slice's
    normaliser. Where one logit exceeds all others by 2^30 in the weights, the normaliser is that
    logit itself (the other weights add less than half an ulp of 1), so the two passes' lse must
    agree bit by bit there."""
    import torch
    import paper_2609_32525_amd as fs
    w = small(f"logits_D{D}_G{G}_N{N}", "f32", D, G, O.MIX_IDENTITY, N=N)
    announce(f"shared logits {w}")
    inp = W.make_inputs(w)
    inp["Ws"] = inp["Ws"] * np.float32(300.0)
    pb, got = run_gpu(w, inp, backward=False)
    a = (np.einsum("bnhd,dg->bhng", inp["x"].astype(np.float64), inp["Ws"].astype(np.float64)) +
         inp["b"]) / inp["tau"].astype(np.float64)[None, :, None, None] / np.log(2.0)
    top = np.sort(a, axis=-1)
    clear = top[..., -1] - top[..., -2] > 30.0
    assert clear.mean() > 0.5
    lse, out = torch.empty_like(pb.lse), torch.empty_like(pb.out)
    fs.deslice_stats_fwd(pb.prob, pb.x, pb.Ws, pb.b, pb.tau, pb.zmix, lse, out)
    torch.cuda.synchronize()
    s, d = pb.lse.cpu().numpy()[clear], lse.cpu().numpy()[clear]
    assert np.array_equal(s, d), f"{(s != d).sum()} of {s.size} normalisers differ"
