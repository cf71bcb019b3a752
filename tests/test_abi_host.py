"""CPU-side checks of the C-ABI library: it loads, exports every function the header declares,
validates arguments before touching the device, and its host-only planner equals the oracle."""
import ctypes
import os
import re

import pytest

import paper_2411_19460_amd as pk
from paper_2411_19460_amd import binding
from oracle import magc_ref

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    text = open(os.path.join(ROOT, "include", "ssd_magc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ssd_\w+|magc_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = binding.lib()
    names = header_functions()
    assert set(names) == set(binding.EXPORTS), names
    for n in names:
        assert getattr(L, n) is not None


def shape(**kw):
    base = dict(dtype=1, nheads=8, headdim=64, ngroups=1, dstate=128, chunk=256, batch=1, seqlen=2048, segment=1024,
                x_batch_stride=0, dt_batch_stride=0, bc_batch_stride=0)
    base.update(kw)
    return pk.ssd_shape_t(**base)


def test_workspace_query_and_shape_validation():
    assert pk.ssd_workspace_bytes(shape(), False) > 0
    assert pk.ssd_workspace_bytes(shape(), True) > pk.ssd_workspace_bytes(shape(), False)
    # workspace follows the segment, not the sequence length: forward exactly; backward up to the two
    # per-chunk partial sums of dA and dD (8 bytes per chunk and head, 256-byte rounding)
    # (compared at the same number of segments in flight: both sequences have at least four segments)
    short, long_ = shape(seqlen=8192, segment=1024), shape(seqlen=1 << 20, segment=1024)
    assert pk.ssd_workspace_bytes(long_, False) == pk.ssd_workspace_bytes(short, False)
    extra = pk.ssd_workspace_bytes(long_, True) - pk.ssd_workspace_bytes(short, True)
    assert 0 <= extra <= 2 * 4 * 8 * ((1 << 20) // 256) + 512
    # a sequence need not be a whole number of segments or chunks: the short tail is read and written in place
    assert 0 < pk.ssd_workspace_bytes(shape(seqlen=2000), True) <= pk.ssd_workspace_bytes(shape(seqlen=2048), True)
    for bad in (dict(dtype=7), dict(nheads=0), dict(segment=1000), dict(ngroups=3),
                dict(chunk=2048), dict(headdim=512), dict(batch=0)):
        assert pk.ssd_workspace_bytes(shape(**bad), True) == 0, bad


@pytest.mark.parametrize("flags", [0, 4, 16])     # 4: shape-generic kernels, 16: fp32 chunk states
@pytest.mark.parametrize("dtype", [0, 1])
def test_scratch_for_the_longest_sequence_serves_every_shorter_one(dtype, flags):
    """Scratch is sized once for the longest sequence of a loop: every shorter one asks for no more, and however many
    segments there are, for no more than four times what one segment asks for, eight times for short segments, and the
    shape-generic kernels for no more than one for long segments (plus what grows with the sequence)."""
    L = binding.lib()
    for heads, groups, chunk, per_seg, batch in ((32, 1, 256, 4, 1), (24, 1, 256, 4, 1), (64, 1, 256, 1, 1), (80, 1, 128, 8, 1), (80, 2, 256, 16, 1),
                                                 (40, 1, 256, 8, 2), (6, 2, 64, 2, 3), (80, 1, 256, 64, 1)):
        segment = chunk * per_seg
        step = max(1, segment // 5)
        for back in (0, 1):
            need = lambda n: L.ssd_workspace_bytes_flags(ctypes.byref(shape(dtype=dtype, nheads=heads, ngroups=groups, batch=batch,  # noqa: E731
                                                                            chunk=chunk, segment=segment, seqlen=n)), back, flags)
            one = need(segment)
            sizes = sorted(set(range(1, 7 * segment, step)) | {k * segment + e for k in range(1, 10) for e in (-1, 0, 1)})
            last = 0
            for n in sizes:
                now = need(n)
                assert now >= last, (heads, chunk, per_seg, back, n, now, last)
                last = now
            short = batch * heads * segment < 163840
            stores = 8 if short else (4 if dtype == 1 and flags != 4 else 1)
            grows = 2 * (-(-sizes[-1] // chunk) * batch * heads * 4 + 256) if back else 2 * (batch * heads * 64 * 128 * 4 + 256)
            assert last <= stores * one + grows, (heads, chunk, per_seg, back, last / one)


def call_fwd(sh, ptrs, ws=0x1000, ws_bytes=1 << 40, flags=0):
    L = binding.lib()
    return L.ssd_fwd(ctypes.byref(sh), *ptrs, ws, ws_bytes, flags, None)


def _device_present():
    import torch
    return torch.cuda.device_count() > 0


@pytest.mark.skipif(_device_present(), reason="feeds fake pointers: every call must be rejected on the host, and is only made where no device could be reached")
def test_fwd_bwd_reject_bad_arguments_before_any_launch():
    # Fake non-NULL pointers: validation must fail before anything dereferences them.
    p = 0x1000
    ok = [p] * 6 + [None, p, p, p]  # x dt A B C D init y final bnd
    assert call_fwd(shape(dtype=9), ok) == -4
    assert call_fwd(shape(segment=1000), ok) == -3
    assert call_fwd(shape(ngroups=3), ok) == -3
    assert call_fwd(shape(nheads=-1), ok) == -2
    assert call_fwd(shape(), [None] + ok[1:]) == -1
    assert call_fwd(shape(), ok, ws=None) == -5
    assert call_fwd(shape(), ok, ws=0x1001) == -5                          # misaligned
    assert call_fwd(shape(), ok, ws_bytes=16) == -5
    assert call_fwd(shape(), ok, flags=1 << 20) == -8
    L = binding.lib()
    okb = [p] * 6 + [None, 0x3000, None, p] + [p] * 6 + [None]    # x dt A B C D init dy dfinal bnd dx ddt dA dB dC dD dinit
    sh = shape()
    assert L.ssd_bwd(ctypes.byref(sh), *okb, 0x1000, 16, 0, None) == -5
    nobnd = list(okb)
    nobnd[9] = None                                                         # checkpoints required when segment < L
    assert L.ssd_bwd(ctypes.byref(sh), *nobnd, 0x1000, 1 << 40, 0, None) == -1
    bad = list(okb)
    bad[10] = None                                                          # dx
    assert L.ssd_bwd(ctypes.byref(sh), *bad, 0x1000, 1 << 40, 0, None) == -1
    alias = list(okb)
    alias[7] = alias[10] = 0x2000                                           # dx aliases dy
    assert L.ssd_bwd(ctypes.byref(sh), *alias, 0x1000, 1 << 40, 0, None) == -8
    assert L.ssd_fwd(None, *ok, 0x1000, 1 << 40, 0, None) == -1
    okd = [p] * 8                                                           # x dt A B C D state y
    assert L.ssd_decode(ctypes.byref(shape(seqlen=3)), *okd[:6], None, p, 0, None) == -1   # state is required
    assert L.ssd_decode(ctypes.byref(shape(seqlen=3, ngroups=3)), *okd, 0, None) == -3
    assert L.ssd_decode(ctypes.byref(shape(seqlen=3, dtype=5)), *okd, 0, None) == -4
    assert L.ssd_decode(ctypes.byref(shape(seqlen=3)), *okd, 2, None) == -8                 # only the residual flag
    assert L.ssd_decode(ctypes.byref(shape(seqlen=0)), *([None] * 8), 0, None) == 0         # nothing to do
    for code in range(-8, 1):
        assert pk.strerror(code) and pk.strerror(code) != "unknown status"
    assert pk.strerror(-99) == "unknown status"


def test_stack_validation():
    sh = shape()
    assert pk.magc_stack_workspace_bytes(sh, 4, 2, True) > pk.magc_stack_workspace_bytes(sh, 4, 2, False) > 0
    assert pk.magc_stack_workspace_bytes(sh, 0, 2, True) == 0
    assert pk.magc_stack_workspace_bytes(shape(x_batch_stride=1 << 30), 4, 2, True) == 0
    assert pk.magc_stack_workspace_bytes(shape(seqlen=2000), 4, 2, True) == 0        # the grid has whole cells only
    assert pk.magc_stack_workspace_bytes(shape(seq_reset=0x1000), 4, 2, True) == 0    # no packed sequences in the stack
    # a larger layer interval keeps more restored activations alive inside a cell
    assert pk.magc_stack_workspace_bytes(sh, 8, 8, True) > pk.magc_stack_workspace_bytes(sh, 8, 2, True)


ERR_NULL, ERR_SHAPE, ERR_DIVISIBILITY, ERR_WORKSPACE, ERR_ARG = -1, -2, -3, -5, -8   # as in include/ssd_magc.h


def test_block_pieces_validate_before_any_launch():
    # every check below fails (or sizes a workspace) on the host; nothing is launched
    L = binding.lib()
    fake = ctypes.c_void_p(0x1000)
    cs = binding.ssd_conv_shape_t(1, 64, 1, 128, 0, 0)
    assert L.ssd_conv1d_workspace_bytes(ctypes.byref(cs)) > 0
    assert L.ssd_conv1d_workspace_bytes(ctypes.byref(binding.ssd_conv_shape_t(7, 64, 1, 128, 0, 0))) == 0      # dtype
    assert L.ssd_conv1d_workspace_bytes(ctypes.byref(binding.ssd_conv_shape_t(1, 64, 1, 128, 0, 32))) == 0     # row stride below C
    assert L.ssd_conv1d_fwd(ctypes.byref(cs), fake, None, None, None, fake, None, None) == ERR_NULL
    ns = binding.ssd_norm_shape_t(1, 64, 4, 1e-5, 128, 0, 0)
    assert L.ssd_gated_norm_workspace_bytes(ctypes.byref(ns)) > 0
    assert L.ssd_gated_norm_workspace_bytes(ctypes.byref(binding.ssd_norm_shape_t(1, 64, 5, 1e-5, 128, 0, 0))) == 0   # 64 % 5
    assert L.ssd_gated_norm_workspace_bytes(ctypes.byref(binding.ssd_norm_shape_t(1, 64, 4, -1.0, 128, 0, 0))) == 0   # eps < 0
    assert L.ssd_gated_norm_fwd(ctypes.byref(binding.ssd_norm_shape_t(1, 64, 4, 1e-5, 128, 32, 0)), fake, fake, fake, fake, None) \
        == ERR_SHAPE                                                                                   # stride below dim
    assert L.ssd_gated_norm_fwd(ctypes.byref(ns), None, fake, fake, fake, None) == ERR_NULL
    assert L.ssd_linear_fwd(16, 12, 8, fake, 0, fake, fake, 0, None) == ERR_DIVISIBILITY             # 12 % 8
    assert L.ssd_linear_fwd(16, 16, 8, fake, 8, fake, fake, 0, None) == ERR_SHAPE                     # stride below in_dim
    assert L.ssd_linear_fwd(16, 16, 8, ctypes.c_void_p(0x1004), 0, fake, fake, 0, None) == ERR_ARG    # alignment
    assert L.ssd_linear_fwd(16, 16, 8, None, 0, fake, fake, 0, None) == ERR_NULL
    assert L.ssd_linear_bwd(16, 16, 8, fake, 0, fake, fake, 0, fake, 0, fake, 64, None) == ERR_ARG    # unknown flag
    bs = binding.magc_block_shape_t(2560, 80, 64, 1, 128, 256, 1e-5, 65536, 4096)
    full = binding.magc_block_shape_t(2560, 80, 64, 1, 128, 256, 1e-5, 65536, 65536)
    w_seg, w_full = (L.magc_block_workspace_bytes(ctypes.byref(x), 1) for x in (bs, full))
    assert 0 < w_seg < w_full / 8                                     # the workspace scales with the segment
    assert L.magc_block_workspace_bytes(ctypes.byref(bs), 0) < w_seg
    assert L.magc_block_workspace_bytes(ctypes.byref(binding.magc_block_shape_t(2560, 4, 64, 1, 128, 256, 1e-5, 1024, 512)), 1) == 0   # H % 8
    assert L.magc_block_workspace_bytes(ctypes.byref(binding.magc_block_shape_t(2560, 80, 64, 1, 128, 256, 1e-5, 1024, 300)), 1) == 0  # segment % chunk
    wide = binding.magc_block_shape_t(64, 8, 8, 1, 520, 64, 1e-5, 70, 128)                               # state wider than the scan takes
    assert L.magc_block_workspace_bytes(ctypes.byref(wide), 0) == 0
    assert L.magc_block_fwd(ctypes.byref(wide), None, fake, None, None, fake, None, None, None, None, fake, 1 << 40, None) == ERR_SHAPE
    par, gr = binding.magc_block_params_t(), binding.magc_block_grads_t()
    assert L.magc_block_fwd(ctypes.byref(bs), ctypes.byref(par), fake, None, None, fake, fake, fake, None, None, fake, 1 << 40, None) == ERR_NULL
    assert L.magc_block_bwd(ctypes.byref(bs), ctypes.byref(par), fake, None, None, fake, None, None, fake, fake, fake, ctypes.byref(gr), None, None, fake, 1 << 40, 0, None) \
        == ERR_NULL
    # the stack: shapes, parameter structs and state arrays are checked before the workspace or a launch
    ss = binding.magc_blockstack_shape_t(bs, 4, 2)
    assert L.magc_blockstack_workspace_bytes(ctypes.byref(ss), 1) > L.magc_blockstack_workspace_bytes(ctypes.byref(ss), 0) > 0
    assert L.magc_blockstack_workspace_bytes(ctypes.byref(binding.magc_blockstack_shape_t(bs, 4, 5)), 0) == 0     # interval above the layer count
    # segments that are walked together are no more than a grid's second dimension counts, however small the block
    tiny = [binding.magc_blockstack_shape_t(binding.magc_block_shape_t(8, 8, 1, 8, 1, 1, 1e-5, n, 1), 1, 1) for n in (200000, 400000)]
    for size in (lambda t: L.magc_blockstack_workspace_bytes(t, 0), lambda t: L.magc_blockstack_workspace_bytes(t, 1),
                 lambda t: L.magc_blockstack_pass_bytes(t, 1, 1 << 60)):
        got = [size(ctypes.byref(t)) for t in tiny]
        assert got[0] == got[1] > 0
    pars = (binding.magc_block_params_t * 4)()
    assert L.magc_blockstack_infer(ctypes.byref(ss), pars, fake, fake, fake, fake, 0, fake, 1 << 40, None) == ERR_NULL      # parameters missing
    for k in binding.BLOCK_PARAMS[:-1]:
        for j in range(4):
            setattr(pars[j], k, 0x1000)
    assert L.magc_blockstack_infer(ctypes.byref(ss), pars, fake, fake, None, fake, 0, fake, 1 << 40, None) == ERR_NULL      # no state array
    assert L.magc_blockstack_infer(ctypes.byref(ss), pars, fake, fake, fake, fake, 0, None, 0, None) == ERR_WORKSPACE
    assert L.magc_blockstack_infer(ctypes.byref(ss), pars, fake, fake, fake, fake, 0, ctypes.c_void_p(0x1010), 1 << 40, None) == ERR_WORKSPACE   # alignment
    assert L.magc_blockstack_infer(ctypes.byref(binding.magc_blockstack_shape_t(bs, 0, 1)), pars, fake, fake, fake, fake, 0, fake, 1 << 40, None) == ERR_SHAPE
    # the pre-norm needs its gradient slot
    grs = (binding.magc_block_grads_t * 1)()
    for k in binding.BLOCK_PARAMS[:-1]:
        setattr(grs[0], "d" + k, 0x1000)
    pars[0].pre_norm_w = 0x1000
    assert L.magc_block_bwd(ctypes.byref(bs), ctypes.byref(pars[0]), fake, None, None, fake, None, None, fake, fake, fake, ctypes.byref(grs[0]), None, None, fake,
                            1 << 40, 64, None) == ERR_ARG       # unknown flag: refused first


CASES = [
    (512, 512, 1, 1, 1, 0, 1, 0, False),
    (4, 1024, 1, 1, 1, 0, 1, 0, False),
    (1024, 4, 1, 1, 1, 0, 1, 0, False),
    (64, 1 << 14, 2560, 671488, 15696, 660736, 256, 0, False),
    (64, 1 << 16, 2560, 671488, 15696, 660736, 256, 0, False),
    (48, 1 << 15, 1024, 269056, 6432, 264448, 256, 0, True),
    (16, 1 << 18, 10240, 2621440, 10240, 20480, 256, 0, False),
    (8, 4096, 10, 1000, 10, 5, 256, 5.0e6, False),
    (8, 4096, 10, 1000, 10, 5, 256, 1.0e12, False),
    (5, 100, 3, 7, 2, 1, 256, 0, False),
    (7, 300, 3, 7, 2, 1, 256, 0, True),
]


@pytest.mark.parametrize("case", CASES)
def test_planner_equals_oracle(case):
    L, S, cl, cs, cg, ct, mult, budget, ic = case
    want = magc_ref.plan(L, S, cl, cs, cg, ct, s_multiple=mult, budget=budget, integer_counts=ic)
    rc, got = pk.magc_plan(L, S, cl, cs, cg, ct, s_multiple=mult, budget=budget, integer_counts=ic)
    assert (got["l"], got["s"]) == (want["l"], want["s"])
    assert got["fits"] == want["fits"] and (rc == 0) == want["fits"]
    for name, w in zip(("m_lckpt", "m_sckpt", "m_grid", "m_state"), want["terms"]):
        assert abs(got[name] - float(w)) <= 1e-12 * max(1.0, float(w))
    assert abs(got["m_total"] - float(want["total"])) <= 1e-12 * float(want["total"])


def test_planner_budget_too_small_and_regimes():
    rc, got = pk.magc_plan(8, 4096, 10, 1000, 10, 5, budget=1.0)
    assert rc == -7 and not got["fits"]
    free = magc_ref.plan(8, 4096, 10, 1000, 10, 5)
    assert (got["l"], got["s"]) == (free["l"], free["s"])
    assert pk.magc_plan(4, 1024, 1, 1, 1, 0)[1]["regime"] == 1     # L^2 <= S
    assert pk.magc_plan(1024, 4, 1, 1, 1, 0)[1]["regime"] == 2     # S^2 <= L
    assert pk.magc_plan(512, 512, 1, 1, 1, 0)[1]["regime"] == 0
    with pytest.raises(pk.SSDError):
        pk.magc_plan(0, 10, 1, 1, 1, 0)
    with pytest.raises(pk.SSDError):
        pk.magc_plan(4, 10, -1, 1, 1, 0)


def test_a_kept_shape_descriptor_is_found_by_value_only():
    """What a first call refuses is refused with the descriptor of an equal number at hand, and a length held in a tensor is read
    on every call."""
    import torch
    x, Bm, seg = torch.empty((1, 48, 2, 8)), torch.empty((1, 48, 1, 8)), torch.tensor(16)
    assert binding._shape_ref(x, Bm, 8, 16, None)[0].segment == 16
    for chunk, segment in ((8.0, 16), (8, 16.0), (8.0, None)):
        with pytest.raises(TypeError):
            binding._shape_ref(x, Bm, chunk, segment, None)
    assert binding._shape_ref(x, Bm, 8, seg, None)[0].segment == 16
    assert binding._shape_ref(x, Bm, 8, seg.add_(8), None)[0].segment == 24


@pytest.mark.parametrize("channels", [1, 2, 3, 4, 5, 255, 256, 257])
def test_convolution_scratch_for_any_number_of_channels(channels):
    """Fewer channels than a thread takes at once make one wave side by side, not none: the division of a launch's waves among the
    runs of tokens has to stand for them too.  Five sums a channel, of at least one workgroup."""
    L = binding.lib()
    for dtype in (0, 1):
        for batch in (1, 3):
            for seqlen in (0, 1, 7, 100, 65536):
                sh = binding.ssd_conv_shape_t(dtype=dtype, channels=channels, batch=batch, seqlen=seqlen, batch_stride=0, u_row_stride=0)
                got = L.ssd_conv1d_workspace_bytes(ctypes.byref(sh))
                assert got >= 5 * channels * 4 and got % 256 == 0, (dtype, batch, seqlen, got)


@pytest.mark.parametrize("channels,batch", [(5376, 1), (10752, 1), (1792, 3), (257, 1), (48, 64), (5377, 300)])
def test_convolution_scratch_of_a_length_does_for_every_shorter_one(channels, batch):
    """A caller sizes one buffer for the longest segment and runs the short last one in it."""
    L = binding.lib()
    most = 0
    for seqlen in range(3000):
        sh = binding.ssd_conv_shape_t(dtype=1, channels=channels, batch=batch, seqlen=seqlen, batch_stride=0, u_row_stride=0)
        got = L.ssd_conv1d_workspace_bytes(ctypes.byref(sh))
        assert got >= most, (seqlen, got, most)
        most = got
