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


@pytest.mark.parametrize("D,G", [(32, 64), (64, 32)])
def test_linearno_backward_keeps_the_column_normaliser_apart(D, G):
    """LinearNO's weights are 2^(t - clse) with clse near 13 at 2^13 points. Subtracted from the
    finished logit it costs one rounding: uniform within 2^-21 for differences up to 16, so a weight
    is off by ln 2 * 2^-21 / sqrt(3) = 1.9e-7 in the mean square, the logit and clse add as much
    each, dz and z a few units of fp32 (4e-7): 6e-7 in all, 8e-7 allowed. As the start value of the
    products it cut every part product at 2^-20 and came to 1.1e-6 and more."""
    from paper_2609_32525_amd.runner import PathBuffers
    from paritycheck import measures
    w = small(f"lno_D{D}_G{G}", "f32", D, G, O.MIX_LINEAR_C, N=1 << 13, B=1, H=2,
              tau_mode="uniform")
    announce(f"linearno normaliser {w}")
    inp, ut = W.make_inputs(w), W.untied_params(w)
    pb = PathBuffers(inp, w.mix, w.dtype, w.eps, untied=ut, linearno=True)
    pb.step()
    got = pb.results()
    prm = {k: inp.get(k) for k in ("A", "Wc", "Wq", "Wk", "Wv", "scale")}
    args = (inp["x"], inp["fx"], inp["Ws"], inp["b"], inp["tau"], ut["Wd"], ut["bd"], ut["taud"],
            w.mix, prm)
    bwd = O.linearno_backward(*args, inp["dout"], fwd=O.linearno_forward(*args))
    bad = {}
    for k in ("dfx", "dWs"):
        n, _ = measures(got[k], bwd[k], 4.0)
        print(f"  {k}: {n:.2e}", flush=True)
        if not n <= 8e-7:
            bad[k] = n
    assert not bad, bad
