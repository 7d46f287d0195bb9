"""Rounding of the token mixes beyond one workgroup, on their own (needs an MI355X): their sums
run in several short chains, since a matrix instruction rounds its running sum."""
import math

import pytest

from paritycheck import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,G,V,bound", [("attn", 64, 64, 1.3e-7), ("linear_c", 512, 16, 6.5e-8)])
def test_mix_sums_in_short_chains(kind, G, V, bound):
    """zmix against 64 bits, normwise over 6 samples (the spread between samples is 1%). u = 6e-8
    is the fp32 unit. linear_c: sums of 16 in four chains of one instruction, joined in two steps,
    and the store: three roundings, u / sqrt(3) each at most, 6.0e-8; one chain of four
    instructions rounds once more on the whole sum (7.3e-8). Attention over nearly equal tokens: the
    product with W_v over 64 columns sets the error, four chains of four instructions
    (1.1e-7) against one of sixteen (1.6e-7)."""
    import torch
    import paper_2609_32525_amd as fs
    announce(f"mix precision {kind} G={G} V={V}")
    B, H = 1, 4
    err = []
    for seed in range(6):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        lim = math.sqrt(6.0 / (2 * V))
        W = [(torch.rand(V, V, device="cuda", generator=g) * 2 - 1) * lim for _ in range(3)]
        z = torch.randn(B, H, G, V, device="cuda", generator=g)
        if kind == "attn":
            z = z * 0.03 + torch.randn(B, H, 1, V, device="cuda", generator=g)
        z = z.contiguous()
        prob = fs.Problem.make(B, 64, H, V, V, G, fs.F32, 1e-5, 0)
        md = fs.MixDesc.make(fs.MIX_ATTN if kind == "attn" else fs.MIX_LINEAR_C, Wc=W[0], Wq=W[0],
                             Wk=W[1], Wv=W[2], scale=1.0 / math.sqrt(V))
        zmix = torch.empty_like(z)
        fs.mix(prob, md, z, zmix, torch.empty(B, H, G, G, device="cuda") if kind == "attn" else None)
        torch.cuda.synchronize()
        zd, Wd = z.double().cpu(), [w.double().cpu() for w in W]
        if kind == "attn":
            P = torch.softmax((zd @ Wd[0]) @ (zd @ Wd[1]).transpose(2, 3) / math.sqrt(V), -1)
            ref = P @ (zd @ Wd[2])
        else:
            ref = zd @ Wd[0]
        err.append(float((zmix.double().cpu() - ref).norm() / ref.norm()))
    mean = sum(err) / len(err)
    print(f"  zmix {mean:.2e}", flush=True)
    assert mean <= bound, err


def test_mix_bwd_alone_stays_a_matrix_product():
    """fs_mix_bwd has no zmix to take the attention's row sums of dP P from; they are formed by
    tile products like the rest: at G = 1024 the call takes 2.5 times the forward's time (21 times
    with a dot product per lane). 8 times allowed."""
    import torch
    import paper_2609_32525_amd as fs
    announce("mix_bwd alone, G=1024")
    B, H, G, V = 1, 8, 1024, 32
    z, dzm = (torch.randn(B, H, G, V, device="cuda") for _ in range(2))
    W = [torch.randn(V, V, device="cuda") / math.sqrt(V) for _ in range(3)]
    prob = fs.Problem.make(B, 64, H, V, V, G, fs.F32, 1e-5, 0)
    md = fs.MixDesc.make(fs.MIX_ATTN, Wq=W[0], Wk=W[1], Wv=W[2], scale=1.0 / math.sqrt(V))
    zmix, dz, P = torch.empty_like(z), torch.empty_like(z), torch.empty(B, H, G, G, device="cuda")
    dm = torch.empty(3 * V * V, device="cuda")
    ws = torch.empty(fs.workspace_bytes(prob, 1), device="cuda", dtype=torch.uint8)

    def us(f):
        f()
        t = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                f()
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) * 100.0)
        return min(t)

    fwd = us(lambda: fs.mix(prob, md, z, zmix, P))
    bwd = us(lambda: fs.mix_bwd(prob, md, z, P, dzm, dz, dm, ws))
    print(f"  forward {fwd:.1f} us, backward {bwd:.1f} us", flush=True)
    assert bwd < 8.0 * fwd


def test_attention_probabilities_are_rounded_once():
    """P = e / L over nearly equal scores: the exponential (an ulp at most, 2^-24 rms over half
    of it), L's rounding, common to a row, and one rounding of the quotient: 2^-24 / sqrt(3)
    each, 4.7e-8 measured with the row's common part, 5.2e-8 allowed. A reciprocal rounded first
    adds another (5.8e-8)."""
    import torch
    import paper_2609_32525_amd as fs
    announce("attention probabilities")
    B, H, G, V = 1, 8, 256, 32
    err = []
    for seed in range(6):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        lim = math.sqrt(6.0 / (2 * V))
        W = [(torch.rand(V, V, device="cuda", generator=g) * 2 - 1) * lim for _ in range(3)]
        z = torch.randn(B, H, G, V, device="cuda", generator=g) * 0.05
        prob = fs.Problem.make(B, 64, H, V, V, G, fs.F32, 1e-5, 0)
        md = fs.MixDesc.make(fs.MIX_ATTN, Wq=W[0], Wk=W[1], Wv=W[2], scale=1.0 / math.sqrt(V))
        zmix, P = torch.empty_like(z), torch.empty(B, H, G, G, device="cuda")
        fs.mix(prob, md, z, zmix, P)
        torch.cuda.synchronize()
        zd, Wd = z.double().cpu(), [w.double().cpu() for w in W]
        ref = torch.softmax((zd @ Wd[0]) @ (zd @ Wd[1]).transpose(2, 3) / math.sqrt(V), -1)
        err.append(float((P.double().cpu() - ref).norm() / ref.norm()))
    mean = sum(err) / len(err)
    print(f"  P {mean:.2e}", flush=True)
    assert mean <= 5.2e-8, err
