"""GPU parity where a kernel's choice of path can go wrong (needs an MI355X): the softmax sums
taken against a reference other than the maximum, fp32 products from bf16 parts, attention among token sets
beyond one workgroup. Same oracle and bar as the parity tests."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paritycheck import Checker, announce
from test_parity_gpu import LN2, compare, run_gpu, small

pytestmark = pytest.mark.gpu


def log2_sums(w, inp, h):
    """log2 of the sums the bf16 passes accept or refuse in head h: against the first slot's
    logit (base 2) brought to within 64 of it."""
    x, Ws = inp["x"][:, :, h].astype(np.float64), inp["Ws"][h].astype(np.float64)
    a = (x @ Ws + inp["b"][h]) / (inp["tau"][h] * LN2)
    top = a.max(-1)
    lse = top + np.log2(np.exp2(a - top[..., None]).sum(-1))
    return lse - (a[..., 0] - np.clip(a[..., 0], -64.0, 64.0))


@pytest.mark.parametrize("D,G", [(16, 32), (32, 64), (64, 64), (32, 256), (16, 1024)])
@pytest.mark.parametrize("b0,side", [(-20.0, "inside"), (-40.0, "inside"), (600.0, "inside"),
                                     (-53.5, "both"), (-600.0, "beyond")])
def test_first_slot_far_off(D, G, b0, side):
    """bf16 sums a point's weights against a reference from its first slot's logit while the sum
    stays below 2^100, and against the maximum where it does not. One head's first slot is set
    b0 / tau off the others: near enough for reference 0 (-20), sums of 2^50 and more that are
    accepted (-40), the first slot far above (600), accepted and refused points in one tile
    (-53.5), every point refused (-600). The other heads are ordinary, so accepted and redone
    tiles meet in one launch."""
    import torch
    import paper_2609_32525_amd as fs
    w = small(f"first_slot_D{D}_G{G}", "bf16", D, G, O.MIX_LINEAR_G, N=333, ws_per_head=True)
    announce(f"first slot {b0} off: {w}")
    inp = W.make_inputs(w)
    inp["b"][1, 0] = b0
    l = log2_sums(w, inp, 1)
    # (1 away from the limit on the sides that must be clear)
    assert {"inside": l.max() < 99.0, "beyond": l.min() > 101.0,
            "both": l.min() < 99.0 and l.max() > 101.0}[side], (l.min(), l.max())
    assert b0 != -40.0 or l.min() > 49.0
    pb, got = run_gpu(w, inp, backward=False)
    ref, _ = O.run_inputs(inp, w.mix, w.eps, backward_too=False)
    c = Checker(f"first_slot/{w.name}/{b0}", "bf16")
    for k in ("z", "s", "zmix", "lse", "out"):
        c.add(k, got[k], ref[k], keep=False)
    lse, out = torch.empty_like(pb.lse), torch.empty_like(pb.out)
    fs.deslice_stats_fwd(pb.prob, pb.x, pb.Ws, pb.b, pb.tau, pb.zmix, lse, out)
    torch.cuda.synchronize()
    c.add("lse(stats)", lse.double().cpu().numpy() * LN2, ref["lse"], keep=False)
    c.add("out(stats)", out.float().cpu().numpy().astype(np.float64), ref["out"], keep=False)
    c.finish()


@pytest.mark.parametrize("D,G", [(32, 64), (16, 32), (32, 256), (16, 1024)])
def test_reference_costs_no_bits(D, G):
    """The reference must not cost the normaliser its last bits: with the first slot 60 below the
    others (base 2) and logits that bf16 operands hold exactly (projections of 8 significant bits,
    tau = log2 e), lse of order 6 to 11 is off by half an ulp (2^-21 = 4.8e-7 at most), by the rounding
    of the running logits and of the projections' two bf16 parts (2^-17 of a part below 2^-8 of the
    logit), of the same size, and by the exponentials', which average out: 7e-7 allowed in the root mean
    square. Differences from the first logit itself are of order 64 to 70 and their sum's logarithm
    rounds at 2^-17: 4e-6."""
    import torch
    import paper_2609_32525_amd as fs
    w = small(f"ref_bits_D{D}_G{G}", "bf16", D, G, O.MIX_IDENTITY, N=2000, H=2, B=1)
    announce(f"reference {w}")
    inp = W.make_inputs(w)
    inp["Ws"] = W.round_to_bf16(inp["Ws"])
    inp["tau"] = np.full(2, 1.0 / LN2, np.float32)
    inp["b"] = np.zeros(G, np.float32)
    inp["b"][0] = -60.0
    pb, got = run_gpu(w, inp, backward=False)
    a = (inp["x"].astype(np.float64).transpose(0, 2, 1, 3) @ inp["Ws"].astype(np.float64) +
         inp["b"]) / (inp["tau"].astype(np.float64)[:, None, None] * LN2)
    ref = a.max(-1) + np.log2(np.exp2(a - a.max(-1)[..., None]).sum(-1))
    lse, out = torch.empty_like(pb.lse), torch.empty_like(pb.out)
    fs.deslice_stats_fwd(pb.prob, pb.x, pb.Ws, pb.b, pb.tau, pb.zmix, lse, out)
    torch.cuda.synchronize()
    e = [float(np.sqrt(np.mean((l.double().cpu().numpy() - ref) ** 2))) for l in (pb.lse, lse)]
    print(f"  lse off by {e[0]:.2e} (slice) {e[1]:.2e} (stats)", flush=True)
    assert max(e) <= 7e-7, e


@pytest.mark.parametrize("D,G", [(32, 64), (32, 48), (64, 32)])
@pytest.mark.parametrize("N", [1, 17, 129, 641])
def test_fp32_parts_ragged(D, G, N):
    """fp32 products from bf16 parts at the edges of their tiles (16 points by 8 wavefronts in
    pass B, 32 by 4 elsewhere)."""
    w = small(f"parts_D{D}_G{G}_N{N}", "f32", D, G, O.MIX_LINEAR_G, N=N)
    announce(f"fp32 parts {w}")
    inp = W.make_inputs(w)
    _, got = run_gpu(w, inp)
    compare(w, inp, got)


@pytest.mark.parametrize("dtype,D,G", [("f32", 16, 128), ("f32", 64, 64), ("bf16", 64, 48),
                                       ("bf16", 32, 80), ("bf16", 16, 272)])
def test_attention_token_sets(dtype, D, G):
    """Attention and its backward with a workgroup per 16 tokens: 3 to 17 blocks, every width,
    the four- and the eight-wavefront forward."""
    w = small(f"attn_{dtype}_D{D}_G{G}", dtype, D, G, O.MIX_ATTN, N=500, H=2)
    announce(f"attention {w}")
    inp = W.make_inputs(w)
    _, got = run_gpu(w, inp)
    compare(w, inp, got)
