"""One generation step for a few sequences at the sizes where its kernels change: two rows (vector ALUs) and three (matrix
cores), widths that are no multiple of a 256-wide piece, two groups whose norms scale the pieces, state rows of more than
128 columns, eight rows per half wave from 768 pairs of head and sequence on, rows of more than 2560 elements, of which
a wave takes two pieces, more partial sums of squares than are asked for ahead.  Checked against the oracle run on each sequence
alone."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import block_ref, linear_ref
from paper_2411_19460_amd import synth
from parity_util import TOL, check, host
from test_gpu_block import BF, F32, dev_bf16, draw, to_dev
from test_gpu_block import test_stack_generation_for_several_sequences_at_once as check_generation
from test_gpu_linear import dev as dev_linear, draw as draw_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    # d_model, H, P, G, N, Q, pre-norm, sequences
    (128, 8, 64, 1, 128, 128, True, 2),
    (320, 8, 64, 1, 128, 128, True, 3),
    (768, 24, 64, 2, 128, 128, True, 12),
    (128, 8, 64, 1, 136, 64, True, 4),
])
def test_generation_rows(shape):
    check_generation(shape)


@pytest.mark.parametrize("shape", [
    # d_model, H, P, G, N, pre-norm, sequences
    (2560, 80, 64, 1, 128, True, 1),     # vector ALUs, the row shared out among the waves, convolution step included
    (2560, 80, 64, 2, 128, True, 2),     # the same for two rows; two groups
    (2560, 80, 64, 1, 128, True, 16),    # eight state rows per half wave; a wave's second piece of k (K = 2560 and 5120)
    (2560, 80, 64, 2, 128, True, 16),    # second pieces scaled by their group's norm
    (768, 24, 64, 1, 128, True, 3),      # 192 partial sums of squares: more than are asked for ahead (160)
    (1024, 32, 64, 1, 128, False, 3),    # 256 of them, no norm in front
    (128, 16, 24, 2, 128, True, 4),      # groups of 192 channels: the convolution step rides, the operand is not packed
    (320, 16, 40, 2, 128, True, 12),     # groups of 320
])
def test_generation_step_from_given_states(shape):
    """One token for each sequence on random states, two layers: output and both states against the oracle run on each sequence
    alone.  Tolerance as for a stack of two layers."""
    dm, H, P, G, N, pre, nseq = shape
    NL, r = 2, np.random.default_rng(78)
    conv_dim = block_ref.dims(None, H, P, G, N)[1]
    layers_h = [draw(60 + j, 1, dm, H, P, G, N, pre)["p"] for j in range(NL)]
    x = BF(r.standard_normal((nseq, dm)) * np.exp(r.uniform(-1.0, 1.0, (nseq, 1))))
    ssm_h, conv_h = F32(r.standard_normal((nseq, NL, H, P, N)) * 0.3), BF(r.standard_normal((nseq, NL, 3, conv_dim)))
    ssm, conv = torch.from_numpy(ssm_h.astype(np.float32)).cuda(), dev_bf16(conv_h)
    out = pk.magc_blockstack_decode(dev_bf16(x), [to_dev(p) for p in layers_h], H, P, G, N, 128, 128, ssm, conv)["out"]
    torch.cuda.synchronize()
    tol = 2 * TOL["bf16"]
    for i in range(nseq):
        fo = block_ref.stack_fwd(x[i:i + 1], layers_h, H, P, G, N, 1e-5, store=synth.round_bf16, conv_states=conv_h[i], ssm_states=ssm_h[i])
        check(f"sequence {i} out", host(out[i:i + 1]), fo["out"], tol)
        for j in range(NL):
            check(f"sequence {i} layer {j} ssm state", host(ssm[i, j]), fo["ssm_states"][j], tol)
            check(f"sequence {i} layer {j} conv state", host(conv[i, j]), fo["conv_states"][j], tol)


@pytest.mark.parametrize("shape", [
    # layers, d_model, H, P, N, sequences
    (3, 2560, 80, 64, 128, 1),   # 242 MB of weights: the last layer's stream
    (3, 2560, 80, 64, 128, 2),
    (3, 2560, 80, 64, 128, 4),   # the same on the matrix cores, rows in three parts
    (3, 2560, 80, 64, 128, 5),   # in two
    (3, 2560, 80, 64, 128, 7),   # and 55 MB of states: they stream in every layer, four rows per half wave
    (3, 2560, 80, 64, 128, 16),  # 126 MB of states, eight rows; rows of the products as they are
    (13, 64, 120, 64, 128, 1),   # 51 MB of states, a row per half wave
    (4, 1024, 32, 64, 256, 8),   # 67 MB of states of 256 columns
    (7, 64, 120, 64, 248, 1),    # 53 MB of states, a row per half wave, the last columns missing
])
def test_generation_step_of_stacks_larger_than_the_cache(shape):
    """Weights and states fetched by streaming loads: output and both states as above."""
    NL, dm, H, P, N, nseq = shape
    r = np.random.default_rng(79)
    conv_dim = block_ref.dims(None, H, P, 1, N)[1]
    layers_h = [draw(60 + j, 1, dm, H, P, 1, N, True)["p"] for j in range(NL)]
    x = BF(r.standard_normal((nseq, dm)))
    ssm_h, conv_h = F32(r.standard_normal((nseq, NL, H, P, N)) * 0.3), BF(r.standard_normal((nseq, NL, 3, conv_dim)))
    ssm, conv = torch.from_numpy(ssm_h.astype(np.float32)).cuda(), dev_bf16(conv_h)
    out = pk.magc_blockstack_decode(dev_bf16(x), [to_dev(p) for p in layers_h], H, P, 1, N, 128, 128, ssm, conv)["out"]
    torch.cuda.synchronize()
    tol = NL * TOL["bf16"]
    for i in range(nseq):
        fo = block_ref.stack_fwd(x[i:i + 1], layers_h, H, P, 1, N, 1e-5, store=synth.round_bf16, conv_states=conv_h[i], ssm_states=ssm_h[i])
        check(f"sequence {i} out", host(out[i:i + 1]), fo["out"], tol)
        for j in range(NL):
            check(f"sequence {i} layer {j} ssm state", host(ssm[i, j]), fo["ssm_states"][j], tol)
            check(f"sequence {i} layer {j} conv state", host(conv[i, j]), fo["conv_states"][j], tol)


@pytest.mark.parametrize("rows", [3, 16])
@pytest.mark.parametrize("K", [2048, 2056, 5120])
def test_products_of_few_long_rows(rows, K):
    """K of eight pieces of 256, of eight and one of eight k, and of twenty: two a wave."""
    x, w, _ = draw_linear(4, rows, K, 136)
    out = pk.ssd_linear_fwd(dev_linear(x), dev_linear(w))
    torch.cuda.synchronize()
    check("out", host(out), linear_ref.linear_fwd(x, w), TOL["bf16"])


def _rounded_products(nseq, d_model, heads, groups):
    """Runs one and two layers; of each layer the share of the input product's stored values (the new row of the convolution
    state) that are not the correctly rounded product of 64 bits.  The first layer reads rows, the second the operand its
    predecessor packed."""
    P, N, g = 64, 128, torch.Generator(device="cuda")
    g.manual_seed(nseq)
    normal = lambda *shape, dtype=torch.float32: torch.randn(shape, generator=g, device="cuda", dtype=dtype)  # noqa: E731
    di = heads * P
    conv, d_in = di + 2 * groups * N, 2 * di + 2 * groups * N + heads
    layers = [{"W_in": normal(d_in, d_model, dtype=torch.bfloat16).mul_(d_model ** -0.5), "conv_w": normal(conv, 4) * 0.5,
               "conv_b": normal(conv) * 0.2, "dt_bias": normal(heads) - 4, "A": -torch.rand(heads, generator=g, device="cuda") * 15 - 1,
               "D": normal(heads), "norm_w": 1 + 0.3 * normal(di), "W_out": normal(d_model, di, dtype=torch.bfloat16).mul_(di ** -0.5),
               "pre_norm_w": 1 + 0.3 * normal(d_model)} for _ in range(2)]
    x0 = normal(nseq, d_model, dtype=torch.bfloat16)
    ssm, cs = normal(nseq, 2, heads, P, N) * 0.3, normal(nseq, 2, 3, conv, dtype=torch.bfloat16)
    one, two = (pk.magc_blockstack_decode(x0, layers[:n], heads, P, groups, N, 64, 64, ssm[:, :n].clone(), c)["out"]
                for n, c in ((1, cs[:, :1].clone()), (2, cs)))
    torch.cuda.synchronize()
    assert two.shape == one.shape
    for j, x in enumerate((x0, one)):
        p, x = layers[j], x.cpu().double()
        u = x * torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-5) * p["pre_norm_w"].cpu().double()
        want = (u @ p["W_in"].cpu().double().T)[:, di:di + conv].to(torch.bfloat16)
        yield float((cs[:, j, 2].cpu() != want).double().mean())


@pytest.mark.parametrize("nseq,d_model,heads,groups", [(2, 320, 8, 1), (3, 320, 8, 1), (8, 1024, 32, 2)])
def test_few_sequences_keep_the_precision_of_the_normalised_operand(nseq, d_model, heads, groups):
    """Up to eight rows the products' operands (the row times the norm's weight) are good to 16 bits, so the rounded product is
    almost always the correctly rounded one: its error before that is at most 2^-18 of the terms' root sum of squares, against
    half an ulp of 2^-9 of the value, and values spread like normals of the same size: about 2^-8 of them (0.4 %) come out one
    step away (with operands rounded to 8 bits: over a quarter)."""
    for off in _rounded_products(nseq, d_model, heads, groups):
        assert off < 0.015


@pytest.mark.parametrize("nseq,d_model,heads,groups", [(1, 1024, 32, 1), (2, 1024, 32, 1), (3, 1024, 32, 1), (4, 1024, 32, 2), (4, 2560, 80, 1)])
def test_up_to_four_sequences_multiply_operands_of_32_bits(nseq, d_model, heads, groups):
    """Up to four rows the operands are fp32 values (on the matrix cores as three bf16 parts of 8 bits each): what is left is the
    rounding of sums of up to 2560 terms in fp32, at most a few 2^-22 of their root sum of squares, so that by the same count
    a few 2^-12 of the values (below 0.1 %) may come out one step away.  Operands of 16 bits miss 0.23-0.3 %."""
    for off in _rounded_products(nseq, d_model, heads, groups):
        print(f"{nseq} rows of {d_model}: {off:.2e} of the products one step away")
        assert off < 1e-3


@pytest.mark.parametrize("nseq", [2, 3, 6, 9])
def test_infinities_pass_through_the_packed_operand(nseq):
    """No norm between the layers: where the first layer's output overflows to an infinity, the second layer's product of it is
    an infinity of the weight's sign, not NaN, however many parts the operand is carried in."""
    H, P, N, dm, g = 8, 64, 128, 512, torch.Generator(device="cuda")
    g.manual_seed(nseq)
    normal = lambda *shape, dtype=torch.float32: torch.randn(shape, generator=g, device="cuda", dtype=dtype)  # noqa: E731
    di, conv = H * P, H * P + 2 * N
    layers = [{"W_in": normal(2 * di + 2 * N + H, dm, dtype=torch.bfloat16).mul_(dm ** -0.5), "conv_w": normal(conv, 4) * 0.5,
               "conv_b": normal(conv) * 0.2, "dt_bias": normal(H) - 4, "A": -torch.rand(H, generator=g, device="cuda") * 15 - 1, "D": normal(H),
               "norm_w": 1 + 0.3 * normal(di), "W_out": normal(dm, di, dtype=torch.bfloat16).mul_(di ** -0.5)} for _ in range(2)]
    layers[0]["W_out"][77] = 0
    layers[0]["W_out"][77, 5], layers[0]["norm_w"][5] = 1e37, 3e3
    x0 = normal(nseq, dm, dtype=torch.bfloat16)
    ssm, cs = normal(nseq, 2, H, P, N) * 0.3, normal(nseq, 2, 3, conv, dtype=torch.bfloat16)
    one = pk.magc_blockstack_decode(x0, layers[:1], H, P, 1, N, 64, 64, ssm[:, :1].clone(), cs[:, :1].clone())["out"]
    pk.magc_blockstack_decode(x0, layers, H, P, 1, N, 64, 64, ssm, cs)
    torch.cuda.synchronize()
    hit = torch.isinf(one[:, 77])
    assert hit.any() and torch.isfinite(one).sum() == one.numel() - hit.sum()
    want = torch.sign(one[:, 77, None].float() * layers[1]["W_in"][di:di + conv, 77].float()) * float("inf")
    assert torch.equal(cs[hit, 1, 2].float(), want[hit])


@pytest.mark.parametrize("nseq", [2, 3, 6, 9])
def test_an_infinite_norm_weight_gives_infinite_products(nseq):
    """The row times the norm's weight overflows in one element: the products are infinities of its weight's sign, not NaN, however
    many parts the operand is carried in."""
    H, P, N, dm, g = 8, 64, 128, 512, torch.Generator(device="cuda")
    g.manual_seed(nseq)
    normal = lambda *shape, dtype=torch.float32: torch.randn(shape, generator=g, device="cuda", dtype=dtype)  # noqa: E731
    di, conv = H * P, H * P + 2 * N
    layer = {"W_in": normal(2 * di + 2 * N + H, dm, dtype=torch.bfloat16).mul_(dm ** -0.5), "conv_w": normal(conv, 4) * 0.5,
             "conv_b": normal(conv) * 0.2, "dt_bias": normal(H) - 4, "A": -torch.rand(H, generator=g, device="cuda") * 15 - 1, "D": normal(H),
             "norm_w": 1 + 0.3 * normal(di), "W_out": normal(dm, di, dtype=torch.bfloat16).mul_(di ** -0.5), "pre_norm_w": 1 + 0.3 * normal(dm)}
    layer["pre_norm_w"][77] = float("inf")
    x0 = normal(nseq, dm, dtype=torch.bfloat16)
    ssm, cs = normal(nseq, 1, H, P, N) * 0.3, normal(nseq, 1, 3, conv, dtype=torch.bfloat16)
    pk.magc_blockstack_decode(x0, [layer], H, P, 1, N, 64, 64, ssm, cs)
    torch.cuda.synchronize()
    want = torch.sign(x0[:, 77, None].float() * layer["W_in"][di:di + conv, 77].float()) * float("inf")
    assert torch.equal(cs[:, 0, 2].float(), want)


def test_parameters_are_checked_on_every_step():
    """A stack that one step accepted is refused once one of its tensors, at the same address, has another shape."""
    from paper_2411_19460_amd import binding
    want = binding._block_layout(torch.empty((1, 128), dtype=torch.bfloat16, device="cuda"), {}, 8, 64, 1, 128, 64, None, 1e-5)[1]
    layers = [{k: torch.zeros(shp, dtype=dty, device="cuda") for k, (shp, dty) in want.items()} for _ in range(2)]
    x = torch.zeros((1, 128), dtype=torch.bfloat16, device="cuda")
    step = lambda: pk.magc_blockstack_infer(x, layers, 8, 64, 1, 128, 64, 64)  # noqa: E731
    step()
    for k in ("W_in", "conv_w", "D"):
        t = layers[1][k]
        layers[1][k].unsqueeze_(0)
        with pytest.raises(ValueError, match=k):
            step()
        t.squeeze_(0)
    step()
    torch.cuda.synchronize()
