"""Products of few rows whose row is longer than the waves of a workgroup take in one turn, and those at the edges of how columns and waves are
shared out: twelve waves and thirteen pieces, workgroups of eight columns where there are many, two even rounds where one round's columns
do not suffice.  Alone, and in a generation step: normalised rows in turns, the packed operand in turns (one norm group and two, whose
norms scale the pieces), several tiles of packed output to a workgroup."""
import numpy as np
import pytest
import torch

import paper_2411_19460_amd as pk
from oracle import block_ref
from paper_2411_19460_amd import synth
from parity_util import TOL, check, host
from test_gpu_block import BF, F32, dev_bf16, draw, to_dev
from test_gpu_generate_rows import test_generation_step_from_given_states as check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,rows", [
    (6136, 136, (1, 2, 3, 16)),     # twelve pieces of 512; twelve waves of two pieces of 256
    (6152, 136, (1, 2, 3, 16)),     # thirteen, in two turns
    (2824, 4104, (1, 2, 3, 8)),     # twelve pieces of 256, one a wave
    (3080, 1032, (3, 16)),          # thirteen: two a wave
    (1032, 16392, (1, 2, 3)),       # eight columns a workgroup, many rounds
    (2568, 16392, (1, 2)),          # the same with one row, more columns with two
    (2824, 16648, (3, 16)),         # two rounds of at most four tiles
    (2312, 24712, (3, 16)),         # of at most six
    (5128, 131080, (2,)),           # of at most 512 columns
])
def test_edges(K, N, rows):
    """Sums in fp32 and one rounding, half an ulp (2^-9 of the value); a reference product in fp32 is off by a few ulps of fp32."""
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    w = torch.randn((N, K), generator=g, device="cuda", dtype=torch.bfloat16) * K ** -0.5
    for r in rows:
        x = torch.randn((r, K), generator=g, device="cuda", dtype=torch.bfloat16)
        out = pk.ssd_linear_fwd(x, w)
        torch.cuda.synchronize()
        want = x.float() @ w.float().T
        worst = ((out.float() - want).abs() / (want.abs() + 1)).max()
        assert worst <= 2 ** -8, (r, worst)


@pytest.mark.parametrize("shape", [
    # d_model, H, P, G, N, pre-norm, sequences
    *((64, 120, 64, G, 128, True, nseq) for G in (1, 2) for nseq in (2, 3, 6, 16)),  # 7680 channels behind the scan, groups of 7680 and 3840
    (3072, 8, 64, 1, 128, True, 3),        # normalised rows over twelve waves
    *((4104, 40, 64, 1, 128, True, nseq) for nseq in (2, 3, 6, 16)),                 # in two turns; 32 columns of packed output a workgroup
])
def test_steps_of_long_rows(shape):
    check_step(shape)


@pytest.mark.parametrize("shape,tokens", [
    ((2560, 80, 64, 1, 128), 3),    # normalised rows of 5120 in two turns, in three parts
    ((2560, 80, 64, 1, 128), 4),
    ((64, 120, 64, 1, 128), 2),     # the vector ALUs in turns
    ((64, 120, 64, 2, 128), 5),     # groups of 3840
])
def test_tokens_of_one_sequence(shape, tokens):
    """A few tokens of one sequence on given states, two layers, against the oracle.  Tolerance as for a stack of two layers."""
    dm, H, P, G, N = shape
    NL, r = 2, np.random.default_rng(81)
    conv_dim = block_ref.dims(None, H, P, G, N)[1]
    layers_h = [draw(60 + j, 1, dm, H, P, G, N, True)["p"] for j in range(NL)]
    x = BF(r.standard_normal((tokens, dm)))
    ssm_h, conv_h = F32(r.standard_normal((NL, H, P, N)) * 0.3), BF(r.standard_normal((NL, 3, conv_dim)))
    st = pk.magc_blockstack_infer(dev_bf16(x), [to_dev(p) for p in layers_h], H, P, G, N, 128, 128,
                                  ssm_state=torch.from_numpy(ssm_h.astype(np.float32)).cuda(), conv_state=dev_bf16(conv_h))
    torch.cuda.synchronize()
    tol = 2 * TOL["bf16"]
    fo = block_ref.stack_fwd(x, layers_h, H, P, G, N, 1e-5, store=synth.round_bf16, conv_states=conv_h, ssm_states=ssm_h)
    check("out", host(st["out"]), fo["out"], tol)
    for j in range(NL):
        check(f"layer {j} ssm state", host(st["ssm_state"][j]), fo["ssm_states"][j], tol)
        check(f"layer {j} conv state", host(st["conv_state"][j]), fo["conv_states"][j], tol)


@pytest.mark.parametrize("K,N,rows", [
    (264, 520, (3, 8, 9)),           # single tiles: two waves of a row, the last of eight elements
    (1024, 40, (3, 4, 5, 8, 9)),     # four waves
    (1032, 32776, (3, 4, 5)),        # five pieces in two turns of three waves
    (2048, 32768, (3, 4)),           # eight waves
    (4104, 32776, (4,)),             # seventeen pieces in five turns
    (7176, 72, (3, 16)),             # two turns of eight waves for twenty-nine pieces, two a wave
    (14336, 72, (3, 16)),            # four turns of seven waves instead of three of ten
    (2568, 16392, (3, 16)),          # eleven pieces: two a wave where twelve waves need a second round
    (6152, 40, (1, 2)),              # the vector ALUs: thirteen pieces in two turns of seven, four columns a workgroup
    (2568, 12296, (2,)),             # two turns of three
    (2560, 12296, (2,)),             # five waves, eight columns
    (8192, 12296, (1, 2)),           # eight waves in two turns, four in four
    (520, 12296, (1, 2)),            # two waves, eight columns for two rows
    (1032, 3592, (1,)),              # one workgroup a unit, of sixteen columns
    (1032, 4104, (1,)),              # of four again
    (1000, 50296, (16,)),            # three tiles of a row in four waves
    (4096, 32776, (8,)),             # eight waves, single tiles
])
def test_products_alone(K, N, rows):
    """Tolerance as above."""
    test_edges(K, N, rows)
