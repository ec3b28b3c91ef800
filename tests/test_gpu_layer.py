"""The pieces composed into one layer, through the C ABI, against the oracle's chain in fp64:
    y = Q(P AdaLN(x)) Q(P^T W)^T + b                       (paper App. C + Eq. 8)
    y = Q(x H P) Q((W H) P)^T                              (paper App. D + Eq. 8)
The quantizer sees bf16 values that can differ from the oracle's by one rounding step on a few
outputs of the normalisation / rotation (see test_gpu_norm.py), so the products are compared with
the tolerance of the product kernel plus the effect of those steps; the Hadamard case also checks the
qualitative claim that rotation plus reorder lowers the layer's output error on outlier-heavy
activations."""
import ctypes
import sys

import numpy as np
import pytest
import torch

from oracle import calib as OC
from oracle import formats as OF
from oracle import gemm as OG
from oracle import hadamard as OH
from oracle import norm as ON
from oracle import quantize as OQ
from paper_2605_09503_amd import pq, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _bits(v):
    return synth.f64_to_bf16_bits(np.asarray(v, dtype=np.float64))


def _dev(bits):
    return pq.bf16_from_bits(bits, DEV)


def _host_bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def _weights_operand(fmt, g, w_bits, perm_d):
    N, K = w_bits.shape
    codes, scales = pq.alloc_quantized(fmt, g, N, K, DEV)
    tw = torch.ones(1, dtype=torch.float32, device=DEV)
    pq.pq_quantize_weights(fmt, g, _dev(w_bits), perm_d, codes, scales, tw)
    return pq.pq_pack_operand(fmt, g, codes, scales), tw


@pytest.mark.parametrize("fmt,g", [(pq.FMT_INT4, 64), (pq.FMT_NVFP4, 16)])
def test_adaln_quantize_gemm_bias_layer(fmt, g):
    M, N, K, per = 96, 72, 768, 40
    _say("layer adaln fmt=%d g=%d" % (fmt, g))
    rng = np.random.default_rng(9990 + fmt)
    chan = np.exp(0.4 * rng.standard_normal(K))
    chan[rng.choice(K, 8, replace=False)] *= 20.0
    x_bits = _bits(rng.standard_normal((M, K)) * chan + 0.2)
    w_bits = _bits(0.03 * rng.standard_normal((N, K)))
    n_mod = -(-M // per)
    s_bits = _bits(0.3 * rng.standard_normal((n_mod, K)))
    b_bits = _bits(0.3 * rng.standard_normal((n_mod, K)))
    bias_bits = _bits(0.5 * rng.standard_normal(N))
    perm = rng.permutation(K).astype(np.int32)
    perm_d = torch.from_numpy(perm).to(DEV)

    # oracle chain
    y_norm = ON.adaln_reordered(OF.bf16_bits_to_f64(x_bits), OF.bf16_bits_to_f64(s_bits), OF.bf16_bits_to_f64(b_bits),
                                per, 1e-6, perm)
    a64 = OF.bf16_bits_to_f64(ON.to_bf16_bits(y_norm))
    w64 = OF.bf16_bits_to_f64(w_bits)[:, perm]
    ta = OQ.nvfp4_tensor_scale(OC.absmax(a64)) if fmt == pq.FMT_NVFP4 else None
    tw = OQ.nvfp4_tensor_scale(OC.absmax(w64)) if fmt == pq.FMT_NVFP4 else None
    qa, qw = OQ.quantize(fmt, g, a64, ta), OQ.quantize(fmt, g, w64, tw)
    y_ref = OG.add_bias(OG.dequant_product(fmt, g, qa, qw), OF.bf16_bits_to_f64(bias_bits))

    # library chain
    Ta = torch.full((1,), float(ta) if ta is not None else 1.0, dtype=torch.float32, device=DEV)
    a_op = pq.pq_norm_quantize_act_packed(pq.NORM_ADALN, fmt, g, _dev(x_bits), 1e-6, Ta, perm_d, None, _dev(s_bits),
                                          _dev(b_bits), per)
    w_op, Tw = _weights_operand(fmt, g, w_bits, perm_d)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    pq.pq_qgemm_packed_bias(fmt, g, a_op, Ta, w_op, Tw, _dev(bias_bits), y, M, N, K)
    torch.cuda.synchronize()
    got = OF.bf16_bits_to_f64(_host_bits(y))
    # one bf16 step on an activation moves it by at most 2^-8 |a|; it reaches the output through at most
    # one quantization step of its group: bound the whole effect by a small multiple of the layer's scale
    scale = np.sqrt(np.mean(y_ref ** 2))
    assert np.abs(got - y_ref).max() <= 0.02 * scale + 2.0 ** -8 * np.abs(y_ref).max()
    assert np.mean(np.abs(got - y_ref) <= 2.0 ** -8 * np.abs(y_ref) + 1e-3 * scale) > 0.99


def test_hadamard_then_reorder_layer_lowers_the_output_error():
    M, N, K, fmt, g = 128, 96, 1024, pq.FMT_INT4, 64
    rng = np.random.default_rng(9995)
    chan = np.exp(0.3 * rng.standard_normal(K))
    chan[rng.choice(K, 6, replace=False)] *= 40.0            # massive outlier channels
    x_bits = _bits(rng.standard_normal((M, K)) * chan)
    w_bits = _bits(0.03 * rng.standard_normal((N, K)))
    x64, w64 = OF.bf16_bits_to_f64(x_bits), OF.bf16_bits_to_f64(w_bits)
    y_true = x64 @ w64.T
    one = torch.ones(1, dtype=torch.float32, device=DEV)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)

    def rel_err(yq):
        return float(np.sum((OF.bf16_bits_to_f64(_host_bits(yq)) - y_true) ** 2) / np.sum(y_true ** 2))

    # plain W4A4
    w_op, _ = _weights_operand(fmt, g, w_bits, None)
    pq.pq_qgemm_packed(fmt, g, pq.pq_quantize_act_packed(fmt, g, _dev(x_bits), one), one, w_op, one, y, M, N, K)
    torch.cuda.synchronize()
    e_plain = rel_err(y)

    # PermuQuant-H: rotate both sides, select the order on the rotated tensors, quantize, multiply
    xr = pq.pq_hadamard_reorder(_dev(x_bits))
    wr = pq.pq_hadamard_reorder(_dev(w_bits))
    sa = torch.zeros(K, dtype=torch.float64, device=DEV)
    sw = torch.zeros(K, dtype=torch.float64, device=DEV)
    pq.pq_calib_moments(xr, sa)
    pq.pq_calib_moments(wr, sw)
    perm_d = torch.empty(K, dtype=torch.int32, device=DEV)
    rep = pq.pq_select_perm(fmt, g, sa, sw, [xr], wr, 1.0, 1.0, perm_d)
    a_op = pq.pq_hadamard_quantize_act_packed(fmt, g, _dev(x_bits), one, perm_d)
    w_codes, w_scales = pq.alloc_quantized(fmt, g, N, K, DEV)
    pq.pq_quantize_weights(fmt, g, wr, perm_d, w_codes, w_scales, torch.ones(1, dtype=torch.float32, device=DEV))
    pq.pq_qgemm_packed(fmt, g, a_op, one, pq.pq_pack_operand(fmt, g, w_codes, w_scales), one, y, M, N, K)
    torch.cuda.synchronize()
    e_h = rel_err(y)
    _say("output error: plain %.4g, Hadamard + reorder %.4g (accepted=%s)" % (e_plain, e_h, rep.accepted))
    assert e_h < 0.75 * e_plain

    # and the oracle's chain gives the same product up to the tolerance of the pieces
    perm = perm_d.cpu().numpy()
    a64 = OF.bf16_bits_to_f64(OH.to_bf16_bits(OH.rotate_reordered(x64, perm)))
    wr64 = OF.bf16_bits_to_f64(OH.to_bf16_bits(OH.rotate(w64)))[:, perm]
    y_ref = OG.dequant_product(fmt, g, OQ.quantize(fmt, g, a64), OQ.quantize(fmt, g, wr64))
    got = OF.bf16_bits_to_f64(_host_bits(y))
    scale = np.sqrt(np.mean(y_ref ** 2))
    assert np.abs(got - y_ref).max() <= 0.03 * scale + 2.0 ** -8 * np.abs(y_ref).max()


def test_forward_path_replays_from_a_captured_graph():
    """The forward entry points allocate nothing and never synchronise, so a caller can capture them in a
    graph: three replays on refreshed inputs, with eager work and synchronisations in between, each equal
    to the eager result bit for bit."""
    M, N, K, fmt, g = 200, 136, 1024, pq.FMT_INT4, 64
    rng = np.random.default_rng(9996)
    perm_d = torch.from_numpy(rng.permutation(K).astype(np.int32)).to(DEV)
    gamma = _dev(_bits(1.0 + 0.2 * rng.standard_normal(K)))
    bias = _dev(_bits(0.5 * rng.standard_normal(N)))
    w_op, Tw = _weights_operand(fmt, g, _bits(0.03 * rng.standard_normal((N, K))), perm_d)
    one = torch.ones(1, dtype=torch.float32, device=DEV)
    x = torch.empty((M, K), dtype=torch.bfloat16, device=DEV)
    a_op = torch.zeros(pq.pq_operand_bytes(fmt, g, M, K), dtype=torch.uint8, device=DEV)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)

    def forward(out):
        pq.pq_norm_quantize_act_packed(pq.NORM_RMS, fmt, g, x, 1e-6, one, perm_d, gamma, operand=a_op)
        pq.pq_qgemm_packed_bias(fmt, g, a_op, one, w_op, Tw, bias, out, M, N, K)

    x.copy_(_dev(_bits(rng.standard_normal((M, K)))))
    forward(y)                                   # warm-up outside the capture (first-use set-up of the kernels)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        forward(y)
    for i in range(3):
        x.copy_(_dev(_bits(rng.standard_normal((M, K)) * (1.0 + i))))
        y_eager = torch.empty_like(y)
        forward(y_eager)
        torch.cuda.synchronize()
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), y_eager.view(torch.int16)), "replay %d differs" % i


@pytest.mark.parametrize("fmt,g,M,N,K,tile", [
    (pq.FMT_NVFP4, 16, 300, 264, 1088, (32, 32)), (pq.FMT_INT4, 64, 520, 200, 1024, (32, 32)),
    (pq.FMT_NVFP4, 16, 4608, 512, 12288, (64, 96)), (pq.FMT_NVFP4, 16, 4608, 3072, 3072, (224, 256)),
    (pq.FMT_INT3, 32, 3600, 4088, 192, (256, 256)), (pq.FMT_INT4, 64, 2344, 3656, 256, (224, 256)),
    (pq.FMT_INT3, 64, 4090, 4088, 320, (256, 256)),
])
def test_forward_path_in_a_hip_graph(fmt, g, M, N, K, tile):
    """The deployment path (activations quantized straight into the GEMM's operand layout, then the product)
    captured into a HIP graph: every replay, with eager work and synchronisations in between, gives the
    bits of the eager run.  Nothing in the two calls allocates, synchronises or clears memory, so they can be
    captured as they are.  (The third shape takes the large-tensor quantizer; the last four the large tiles of the two
    product kernels.)"""
    assert pq.pq_qgemm_tile(fmt, g, M, N, K) == tile, "this shape is here for the tile it takes: choose another"
    _say("forward path in a graph fmt=%d g=%d %dx%dx%d" % (fmt, g, M, N, K))
    rng = np.random.default_rng(9970 + g + M)
    x = _dev(_bits(rng.standard_normal((M, K)) * np.exp(0.5 * rng.standard_normal(K))))
    w_op, tw = _weights_operand(fmt, g, _bits(0.02 * rng.standard_normal((N, K))), None)
    ta = torch.full((1,), 0.002, dtype=torch.float32, device=DEV)
    a_op = torch.zeros(pq.pq_operand_bytes(fmt, g, M, K), dtype=torch.uint8, device=DEV)   # alignment gaps stay zero
    y_eager = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    pq.pq_quantize_act_packed(fmt, g, x, ta, a_op)
    pq.pq_qgemm_packed(fmt, g, a_op, ta, w_op, tw, y_eager, M, N, K)
    torch.cuda.synchronize()
    a_eager = a_op.clone()
    y = torch.empty_like(y_eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pq.pq_quantize_act_packed(fmt, g, x, ta, a_op)
        pq.pq_qgemm_packed(fmt, g, a_op, ta, w_op, tw, y, M, N, K)
    for replay in range(3):
        a_op.zero_()
        y.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(a_op, a_eager), "operand of replay %d differs" % replay
        assert torch.equal(y.view(torch.int16), y_eager.view(torch.int16)), "output of replay %d differs" % replay
        # eager use of the same buffers between the replays
        pq.pq_quantize_act_packed(fmt, g, x, ta, a_op)
        torch.cuda.synchronize()


class _Asked:
    """A tensor that is only reached through its methods."""
    def __init__(self, t):
        self.t = t
        self.shape = t.shape

    device = property(lambda self: self.t.device)

    def data_ptr(self):
        return self.t.data_ptr()

    def stride(self, d):
        return self.t.stride(d)

    def numel(self):
        return self.t.numel()


@pytest.mark.parametrize("wrap", [lambda t: t, torch.nn.Parameter, _Asked])
@pytest.mark.parametrize("fmt,g", [(pq.FMT_NVFP4, 16), (pq.FMT_INT4, 64)])
def test_calls_by_position_by_name_and_on_another_stream(fmt, g, wrap):
    # the natively marshalled calls: positions and names, tensors and what behaves like one, buffers given and made, the
    # stream that is current
    M, N, K = 33, 72, 192
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16)
    hold = (lambda t: t) if wrap is torch.nn.Parameter else wrap       # a Parameter holds floating point only
    x, w, bias = rnd(M, K), rnd(N, K), rnd(N)
    tx, tw = torch.full((1,), 0.002, device=DEV), torch.empty(1, device=DEV)
    wc, ws = pq.alloc_quantized(fmt, g, N, K, DEV)
    pq.pq_quantize_weights(fmt, g, w, None, wc, ws, tw)
    wo = pq.pq_pack_operand(fmt, g, wc, ws)
    ac, asc = pq.alloc_quantized(fmt, g, M, K, DEV)
    want = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    pq.pq_quantize_act(fmt, g, x, None, tx, ac, asc)
    pq.pq_qgemm(fmt, g, ac, asc, tx, wc, ws, tw, want)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side), torch.no_grad():
        torch.cuda._sleep(1000000)                       # what runs on another stream would be early
        xs = torch.empty_like(x)
        xs.copy_(x)
        bc, bs = pq.alloc_quantized(fmt, g, M, K, DEV)
        pq.pq_quantize_act(fmt, group=g, x=wrap(xs), perm=None, tensor_scale=hold(tx), codes=hold(bc), scales=hold(bs))
        y, yb = (torch.empty_like(want) for _ in range(2))
        yf = torch.empty((M, N), dtype=torch.float32, device=DEV)
        y2 = torch.empty_like(want)
        work = torch.empty(max(16, pq.pq_workspace_bytes(pq.OP_QGEMM, fmt, g, M, N, K)), dtype=torch.uint8, device=DEV)
        pq.pq_qgemm(fmt, g, hold(bc), hold(bs), tx, hold(wc), hold(ws), tw, wrap(y), workspace=hold(work))
        a = pq.pq_quantize_act_packed(fmt, g, wrap(xs), tx)
        mine = torch.empty_like(a)
        given = hold(mine)
        assert pq.pq_quantize_act_packed(fmt, g, wrap(xs), tx, operand=given) is given
        pq.pq_qgemm_packed(fmt, g, hold(a), tx, hold(wo), tw, wrap(y2), M, N, K)
        pq.pq_qgemm_packed_bias(fmt, g, a, tx, wo, tw, wrap(bias), y=wrap(yb), M=M, N=N, K=K, ldy=N)
        pq.pq_qgemm_packed_f32(fmt, g, a, tx, wo, tw, wrap(yf), M, N, K)
        n = pq.pq_norm_quantize_act_packed(pq.NORM_RMS, fmt, g, wrap(xs), 1e-6, tx, gamma=wrap(rnd(K)), K=K)
        sums = [torch.zeros(K, dtype=torch.float64, device=DEV) for _ in range(2)]
        pq.pq_calib_moments(wrap(xs), wrap(sums[0]))
        pq.pq_calib_moments(xs, sums[1], absmax=None, rows=M, K=K, ld=K)
    side.synchronize()
    assert torch.equal(bc, ac) and torch.equal(bs, asc) and torch.equal(mine, a) and n.numel() == a.numel()
    assert torch.equal(y, want) and torch.equal(y2, want) and torch.equal(yf.to(torch.bfloat16), want)
    assert torch.equal(sums[0], sums[1]) and torch.equal(sums[0], x.double().square().sum(0))
    assert (yb.float() - want.float() - bias.float()).abs().max() <= 2.0 ** -7 * (want.float().abs().max() + 4)
    with pytest.raises(pq.PQError) as e:
        pq.pq_qgemm_packed(fmt, g, a, tx, wo, tw, y2, M, N, K, ldy=N - 1)
    assert e.value.code == -2 and "ldy" in str(e.value)
    with pytest.raises(IndexError):
        pq.pq_quantize_act_packed(fmt, g, bias, tx)


def _plain_binding(tmp_path):
    """pq.py beside the library alone: its nine hot calls go through ctypes."""
    import importlib.util
    import os
    import shutil
    (tmp_path / "lib").mkdir()
    os.symlink(pq.lib_path(), tmp_path / "lib" / "libpermuquant.so")
    shutil.copy(pq.__file__, tmp_path / "plain_pq.py")
    spec = importlib.util.spec_from_file_location("plain_pq", tmp_path / "plain_pq.py")
    mod = importlib.util.module_from_spec(spec)
    sys.modules["plain_pq"] = mod                        # dataclasses look their module up
    try:
        with pytest.warns(RuntimeWarning, match="native binding"):
            spec.loader.exec_module(mod)
    finally:
        del sys.modules["plain_pq"]
    return mod


@pytest.mark.parametrize("fmt,g", [(pq.FMT_NVFP4, 16), (pq.FMT_INT4, 64)])
def test_calls_without_the_native_binding_give_the_same(tmp_path, fmt, g):
    import inspect
    plain = _plain_binding(tmp_path)
    assert inspect.isbuiltin(pq.pq_qgemm) and inspect.isfunction(plain.pq_qgemm)
    M, N, K = 33, 72, 192
    out = []
    for mod, integer in ((pq, int), (pq, np.int64), (plain, int), (plain, np.int64)):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(5)
        rnd = lambda *s: torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16)
        x, w, bias, gamma = rnd(M, K), rnd(N, K), rnd(N), rnd(K)
        tx, tw = torch.full((1,), 0.002, device=DEV), torch.empty(1, device=DEV)
        wc, ws = pq.alloc_quantized(fmt, g, N, K, DEV)
        pq.pq_quantize_weights(fmt, g, w, None, wc, ws, tw)
        wo = pq.pq_pack_operand(fmt, g, wc, ws)
        ac, asc = pq.alloc_quantized(fmt, g, M, K, DEV)
        y, yp, yb = (torch.empty((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(3))
        yf = torch.empty((M, N), dtype=torch.float32, device=DEV)
        sums = torch.zeros(K, dtype=torch.float64, device=DEV)
        fi, gi, m, n, k = (integer(v) for v in (fmt, g, M, N, K))
        mod.pq_quantize_act(fi, gi, x, None, tx, ac, asc, M=m, K=k, ld=k)
        a, norm, had = (torch.zeros(pq.pq_operand_bytes(fmt, g, M, K), dtype=torch.uint8, device=DEV) for _ in range(3))
        assert mod.pq_quantize_act_packed(fi, gi, x, tx).numel() == a.numel()
        assert mod.pq_quantize_act_packed(fi, gi, x, tx, operand=a, K=k) is a
        mod.pq_norm_quantize_act_packed(integer(pq.NORM_RMS), fi, gi, x, 1e-6, tx, gamma=gamma, rows_per_mod=m, operand=norm, K=k)
        mod.pq_hadamard_quantize_act_packed(fi, gi, x, tx, operand=had, K=k)
        mod.pq_qgemm(fi, gi, ac, asc, tx, wc, ws, tw, y, M=m, N=n, K=k, ldy=n)
        mod.pq_qgemm_packed(fi, gi, a, tx, wo, tw, yp, m, n, k, ldy=n)
        mod.pq_qgemm_packed_f32(fi, gi, a, tx, wo, tw, yf, m, n, k)
        mod.pq_qgemm_packed_bias(fi, gi, a, tx, wo, tw, bias, yb, m, n, k)
        mod.pq_calib_moments(x, sums, rows=m, K=k, ld=k)
        torch.cuda.synchronize()
        out.append((ac, asc, a, norm, had, y, yp, yf, yb, sums))
    for other in out[1:]:
        for u, v in zip(out[0], other):
            assert torch.equal(u, v)


class _KernelNode(ctypes.Structure):
    """hipKernelNodeParams"""
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _launches(call):
    """Threads of a workgroup of each kernel that a call launches: the nodes of the graph it is captured into."""
    call()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    lib, n, threads = pq.load(), ctypes.c_size_t(), []
    lib.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    lib.hipGraphKernelNodeGetParams.argtypes = [ctypes.c_void_p, ctypes.POINTER(_KernelNode)]
    assert lib.hipGraphGetNodes(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert lib.hipGraphGetNodes(graph.raw_cuda_graph(), nodes, ctypes.byref(n)) == 0
    for node in nodes:
        params = _KernelNode()
        assert lib.hipGraphKernelNodeGetParams(node, ctypes.byref(params)) == 0
        threads.append(params.block[0] * params.block[1] * params.block[2])
    return threads


def _dequantized(fmt, g, x, T):
    """Q(x) of the library's own quantizer in 64 bits, from its stored codes and scales."""
    codes, scales = pq.alloc_quantized(fmt, g, x.shape[0], x.shape[1], DEV)
    pq.pq_quantize_act(fmt, g, x, None, T, codes, scales)
    c = torch.stack((codes & 15, codes >> 4), 2).reshape(x.shape).long()
    if fmt == pq.FMT_NVFP4:
        v = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64, device=DEV)[c]
        s = scales.view(torch.float8_e4m3fn).double() * T.double()
    else:
        v, s = (c - 16 * (c > 7).long()).double(), scales.double()
    return codes, scales, v * s.repeat_interleave(g, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,g,M,N,K,tile,waves", [
    # every tile of NVFP4, of groups of 32, and of the larger groups of INT4 and INT3
    (pq.FMT_NVFP4, 16, 61, 1001, 1184, (32, 32), 8), (pq.FMT_NVFP4, 16, 500, 1021, 320, (64, 32), 8),
    (pq.FMT_NVFP4, 16, 449, 3077, 96, (64, 64), 4), (pq.FMT_NVFP4, 16, 227, 2235, 1792, (64, 64), 8),
    (pq.FMT_NVFP4, 16, 527, 2569, 96, (64, 96), 4), (pq.FMT_NVFP4, 16, 279, 3495, 1792, (64, 96), 8),
    (pq.FMT_NVFP4, 16, 2309, 3077, 96, (128, 128), 4), (pq.FMT_NVFP4, 16, 4099, 5125, 320, (128, 128), 4),
    (pq.FMT_NVFP4, 16, 2339, 3745, 160, (224, 256), 8), (pq.FMT_NVFP4, 16, 3600, 4081, 160, (256, 256), 8),
    (pq.FMT_INT3, 32, 33, 137, 96, (32, 32), 8), (pq.FMT_INT4, 32, 500, 1021, 1632, (64, 32), 8), (pq.FMT_INT3, 32, 449, 3077, 1184, (64, 64), 4),
    (pq.FMT_INT4, 32, 133, 3735, 2560, (64, 64), 8), (pq.FMT_INT3, 32, 2373, 425, 96, (64, 96), 4), (pq.FMT_INT4, 32, 1159, 837, 2560, (64, 96), 8),
    (pq.FMT_INT3, 32, 4099, 5125, 320, (128, 128), 4), (pq.FMT_INT4, 32, 2101, 3921, 96, (224, 256), 8), (pq.FMT_INT3, 32, 2344, 4081, 192, (224, 256), 8),
    (pq.FMT_INT3, 32, 3600, 4082, 192, (256, 256), 8),
    (pq.FMT_INT4, 64, 77, 1001, 1152, (32, 32), 8), (pq.FMT_INT4, 64, 65, 2915, 64, (64, 32), 8), (pq.FMT_INT4, 64, 1100, 4099, 128, (64, 64), 4),
    (pq.FMT_INT4, 64, 161, 3039, 2560, (64, 64), 8), (pq.FMT_INT4, 64, 2375, 457, 384, (64, 96), 4), (pq.FMT_INT4, 64, 539, 1865, 2560, (64, 96), 8),
    (pq.FMT_INT4, 64, 2345, 833, 64, (128, 128), 4), (pq.FMT_INT4, 64, 2309, 5125, 128, (224, 256), 8), (pq.FMT_INT4, 64, 3600, 4081, 192, (256, 256), 8),
    (pq.FMT_INT3, 128, 100, 300, 256, (32, 32), 8), (pq.FMT_INT3, 64, 65, 2881, 64, (64, 32), 8), (pq.FMT_INT3, 64, 153, 4009, 64, (64, 64), 4),
    (pq.FMT_INT3, 64, 449, 3077, 3072, (64, 64), 4), (pq.FMT_INT3, 64, 1000, 3077, 512, (64, 64), 4), (pq.FMT_INT3, 64, 1889, 1607, 64, (64, 96), 4), (pq.FMT_INT3, 64, 585, 3289, 64, (128, 128), 4),
    (pq.FMT_INT3, 64, 2309, 5125, 128, (224, 256), 8), (pq.FMT_INT3, 64, 3600, 4081, 192, (256, 256), 8),
    # waves that have one step, two, an odd number of them, none; a last step of 32 k
    (pq.FMT_NVFP4, 16, 61, 1001, 32, (32, 32), 8), (pq.FMT_NVFP4, 16, 61, 1001, 512, (32, 32), 8), (pq.FMT_NVFP4, 16, 61, 1001, 544, (32, 32), 8),
    (pq.FMT_NVFP4, 16, 500, 1021, 1056, (64, 32), 8), (pq.FMT_NVFP4, 16, 500, 1021, 1120, (64, 32), 8), (pq.FMT_NVFP4, 16, 449, 3077, 288, (64, 64), 4),
    (pq.FMT_NVFP4, 16, 449, 3077, 864, (64, 64), 4), (pq.FMT_NVFP4, 16, 512, 1650, 3104, (64, 64), 8), (pq.FMT_INT3, 64, 512, 3072, 3136, (64, 96), 8)])
def test_row_and_column_factors_and_bias_of_every_tile(fmt, g, M, N, K, tile, waves):
    """Rows and columns of very different size, a bias, ragged edges: every tile's epilogue takes its own factors.  The
    fp32 product against the 64-bit product of what the quantizer stored: K roundings of 2^-24 of the magnitudes (the INT
    factors h / Q are rounded once more each); the bf16 one with the bias is the fp32 one plus the bias, rounded once."""
    assert pq.pq_qgemm_tile(fmt, g, M, N, K) == tile, "this shape is here for its tile: choose another"
    gen = torch.Generator(device=DEV).manual_seed(M + N + K + g)
    rnd = lambda *s: torch.randn(s, generator=gen, device=DEV)
    rows, cols = torch.arange(M, device=DEV), torch.arange(N, device=DEV)
    x = (rnd(M, K) * torch.exp2((rows % 11 - 5).float())[:, None]).to(torch.bfloat16)
    w = (rnd(N, K) * torch.exp2((cols % 13 - 6).float())[:, None]).to(torch.bfloat16)
    bias = rnd(N).to(torch.bfloat16)
    Ta, Tw = ((t.float().abs().max() / 2688).reshape(1) for t in (x, w))
    _, _, xq = _dequantized(fmt, g, x, Ta)
    wc, ws, wq = _dequantized(fmt, g, w, Tw)
    a, wo = pq.pq_quantize_act_packed(fmt, g, x, Ta), pq.pq_pack_operand(fmt, g, wc, ws)
    ldy = (N + 7) // 8 * 8
    yf = torch.empty((M, ldy), dtype=torch.float32, device=DEV)
    yb = torch.empty((M, ldy), dtype=torch.bfloat16, device=DEV)
    y = torch.empty((M, ldy), dtype=torch.bfloat16, device=DEV)
    pq.pq_qgemm_packed_f32(fmt, g, a, Ta, wo, Tw, yf, M, N, K, ldy=ldy)
    pq.pq_qgemm_packed_bias(fmt, g, a, Ta, wo, Tw, bias, yb, M, N, K, ldy=ldy)
    [threads] = _launches(lambda: pq.pq_qgemm_packed(fmt, g, a, Ta, wo, Tw, y, M, N, K, ldy=ldy))
    assert threads == waves * 64, "this shape is here for the waves that share its tile: choose another"
    yf, yb, y = yf[:, :N], yb[:, :N], y[:, :N]
    bound = (K + 4) * 2.0 ** -24 * (xq.abs() @ wq.abs().t())
    assert ((yf.double() - xq @ wq.t()).abs() <= bound).all()
    assert torch.equal(y, yf.to(torch.bfloat16))
    assert torch.equal(yb, (yf + bias.float()).to(torch.bfloat16))


def _int_operand(fmt, g, rows, K, gen, odd_codes):
    """Row-major codes and scales of the quantizers' form fl32(h / Q), with rows of very different size, zero groups and a
    zero row; odd_codes: nibbles that the quantizers do not write, in some rows."""
    h = torch.exp2(torch.randint(-30, 30, (rows, 1), generator=gen, device=DEV).float()) * \
        (torch.rand((rows, K // g), generator=gen, device=DEV) + 2.0 ** -12).to(torch.bfloat16).float()
    h[torch.rand((rows, K // g), generator=gen, device=DEV) < 0.05] = 0.0
    h[rows // 2] = 0.0
    h = h.to(torch.bfloat16)
    Q = 7 if fmt == pq.FMT_INT4 else 3
    z = torch.randint(-Q, Q + 1, (rows, K), generator=gen, device=DEV)
    if odd_codes:
        z[::3] = torch.randint(-8, 8, z[::3].shape, generator=gen, device=DEV)
    z &= 15
    return (z[:, 0::2] | z[:, 1::2] << 4).to(torch.uint8).contiguous(), (h.double() / Q).float()


@pytest.mark.parametrize("odd_codes", [False, True])
@pytest.mark.parametrize("fmt,g,M,N,K,launches", [
    (pq.FMT_INT4, 32, 1, 128, 32, 1), (pq.FMT_INT4, 32, 77, 1000, 1184, 1), (pq.FMT_INT4, 32, 33, 257, 4096, 1), (pq.FMT_INT4, 64, 31, 45, 64, 1),
    (pq.FMT_INT4, 64, 500, 1021, 1088, 1), (pq.FMT_INT4, 128, 77, 1000, 1152, 1), (pq.FMT_INT4, 256, 300, 900, 512, 1),
    (pq.FMT_INT4, 32, 500, 1021, 2048, 1), (pq.FMT_INT3, 32, 61, 1001, 544, 1), (pq.FMT_INT3, 64, 61, 1001, 8192, 2),
    (pq.FMT_INT3, 128, 300, 900, 640, 1), (pq.FMT_INT3, 64, 500, 1021, 4096, 2), (pq.FMT_INT4, 64, 61, 1001, 8256, 2),
    # one tile more than 256, of 32 and of 64 rows
    (pq.FMT_INT4, 64, 32, 8193, 256, 2), (pq.FMT_INT3, 64, 16, 8225, 256, 2), (pq.FMT_INT3, 64, 97, 4097, 128, 2)])
def test_scales_prepared_in_the_product_kernel(fmt, g, M, N, K, launches, odd_codes):
    """pq_qgemm prepares the scales of small products inside the product kernel (one launch); pq_qgemm_prep and _run keep the
    launch for it.  The same bits, on either side of the lines between the two, and those of the packed operands."""
    gen = torch.Generator(device=DEV).manual_seed(M + N + K + g + odd_codes)
    ac, as_ = _int_operand(fmt, g, M, K, gen, odd_codes)
    wc, ws = _int_operand(fmt, g, N, K, gen, odd_codes)
    ldy = (N + 7) // 8 * 8
    ys = [torch.full((M, ldy), 3.0, dtype=t, device=DEV) for t in (torch.bfloat16, torch.bfloat16, torch.bfloat16, torch.float32, torch.float32)]
    work = torch.empty(max(16, pq.pq_workspace_bytes(pq.OP_QGEMM, fmt, g, M, N, K)), dtype=torch.uint8, device=DEV)
    pq.pq_qgemm(fmt, g, ac, as_, None, wc, ws, None, ys[0], workspace=work, N=N, ldy=ldy)
    assert len(_launches(lambda: pq.pq_qgemm(fmt, g, ac, as_, None, wc, ws, None, ys[0], workspace=work, N=N, ldy=ldy))) == launches
    pq.pq_qgemm_prep(fmt, g, as_, ws, M, N, K, work)
    pq.pq_qgemm_run(fmt, g, ac, as_, None, wc, ws, None, ys[1], work, N=N, ldy=ldy)
    a, w = pq.pq_pack_operand(fmt, g, ac, as_), pq.pq_pack_operand(fmt, g, wc, ws)
    pq.pq_qgemm_packed(fmt, g, a, None, w, None, ys[2], M, N, K, ldy=ldy)
    pq.pq_qgemm_f32(fmt, g, ac, as_, None, wc, ws, None, ys[3], workspace=work, N=N, ldy=ldy)
    pq.pq_qgemm_packed_f32(fmt, g, a, None, w, None, ys[4], M, N, K, ldy=ldy)
    bits = [y.view(torch.int16 if y.dtype == torch.bfloat16 else torch.int32) for y in ys]
    assert torch.equal(bits[0], bits[1]) and torch.equal(bits[0], bits[2]) and torch.equal(bits[3], bits[4])
    assert (ys[0][:, N:] == 3.0).all()


@pytest.mark.parametrize("fmt,g,M,N,K", [
    (pq.FMT_INT4, 32, 1, 128, 32), (pq.FMT_INT4, 32, 33, 257, 4096), (pq.FMT_INT4, 64, 500, 1021, 1088), (pq.FMT_INT3, 32, 61, 1001, 544),
    (pq.FMT_INT3, 64, 61, 1001, 8192), (pq.FMT_INT3, 64, 500, 1021, 4096), (pq.FMT_INT4, 64, 61, 1001, 8256), (pq.FMT_INT3, 64, 512, 3072, 3136)])
def test_a_product_leaves_the_workspace_ready_for_the_run(fmt, g, M, N, K):
    """pq_qgemm == pq_qgemm_prep + pq_qgemm_run with the same workspace: after pq_qgemm, wherever it prepared the scales,
    pq_qgemm_run multiplies with what it left, also other codes of the same scales.  The workspace starts as NaNs."""
    gen = torch.Generator(device=DEV).manual_seed(M + N + K + g)
    ac, as_ = _int_operand(fmt, g, M, K, gen, False)
    wc, ws = _int_operand(fmt, g, N, K, gen, False)
    ldy = (N + 7) // 8 * 8
    work = torch.full((pq.pq_workspace_bytes(pq.OP_QGEMM, fmt, g, M, N, K),), 0xFF, dtype=torch.uint8, device=DEV)
    prepared = work.clone()
    y, again, want = (torch.full((M, ldy), 3.0, dtype=torch.bfloat16, device=DEV) for _ in range(3))
    pq.pq_qgemm(fmt, g, ac, as_, None, wc, ws, None, y, workspace=work, N=N, ldy=ldy)
    pq.pq_qgemm_prep(fmt, g, as_, ws, M, N, K, prepared)
    for codes in (ac, ac.flip(0).contiguous()):
        pq.pq_qgemm_run(fmt, g, codes, as_, None, wc, ws, None, again, work, N=N, ldy=ldy)
        pq.pq_qgemm_run(fmt, g, codes, as_, None, wc, ws, None, want, prepared, N=N, ldy=ldy)
        assert torch.equal(again.view(torch.int16), want.view(torch.int16))
        if codes is ac:
            assert torch.equal(again.view(torch.int16), y.view(torch.int16))
    assert torch.equal(work, prepared)


@pytest.mark.parametrize("fmt,g,M,N,K,tile,launches", [
    (pq.FMT_INT4, 32, 77, 1000, 5120, (32, 32), 1), (pq.FMT_INT4, 32, 77, 1000, 5152, (32, 32), 2),
    (pq.FMT_INT4, 64, 61, 1001, 5376, (32, 32), 2), (pq.FMT_INT4, 64, 61, 1001, 5440, (32, 32), 1),
    (pq.FMT_INT4, 64, 61, 1001, 8192, (32, 32), 2), (pq.FMT_INT4, 64, 61, 1001, 8256, (32, 32), 2),
    (pq.FMT_INT3, 64, 20, 5500, 5376, (32, 32), 2), (pq.FMT_INT3, 64, 20, 5600, 5376, (32, 32), 1), (pq.FMT_INT4, 64, 20, 5600, 5376, (32, 32), 2),
    (pq.FMT_INT4, 64, 500, 1021, 2304, (64, 32), 1), (pq.FMT_INT4, 64, 500, 1021, 2560, (64, 32), 2),
    (pq.FMT_INT4, 64, 500, 1021, 3008, (64, 32), 1), (pq.FMT_INT4, 64, 500, 1021, 3136, (64, 32), 2),
    (pq.FMT_INT3, 64, 500, 1021, 2560, (64, 32), 2), (pq.FMT_INT3, 64, 500, 1021, 3136, (64, 32), 1),
    (pq.FMT_INT4, 64, 32, 8192, 256, (32, 32), 1), (pq.FMT_INT4, 64, 32, 8193, 256, (32, 32), 2),
    (pq.FMT_INT4, 64, 400, 1600, 256, (64, 64), 2), (pq.FMT_NVFP4, 16, 77, 1000, 1152, (32, 32), 1)])
def test_which_products_prepare_their_scales(fmt, g, M, N, K, tile, launches):
    """Either side of each line beyond which a launch prepares the scales: in K, in groups, in tiles and their size, and in
    the codes that the launch would read."""
    assert pq.pq_qgemm_tile(fmt, g, M, N, K) == tile
    gen = torch.Generator(device=DEV).manual_seed(M + N + K + g)
    x, w = (torch.randn((n, K), generator=gen, device=DEV).to(torch.bfloat16) for n in (M, N))
    T = torch.full((1,), 2.0 ** -9, device=DEV)
    (ac, as_), (wc, ws) = (pq.alloc_quantized(fmt, g, n, K, DEV) for n in (M, N))
    pq.pq_quantize_act(fmt, g, x, None, T, ac, as_)
    pq.pq_quantize_act(fmt, g, w, None, T, wc, ws)
    y = torch.empty((M, (N + 7) // 8 * 8), dtype=torch.bfloat16, device=DEV)
    work = torch.empty(max(16, pq.pq_workspace_bytes(pq.OP_QGEMM, fmt, g, M, N, K)), dtype=torch.uint8, device=DEV)
    assert len(_launches(lambda: pq.pq_qgemm(fmt, g, ac, as_, T, wc, ws, T, y, workspace=work, N=N, ldy=y.shape[1]))) == launches


@pytest.mark.parametrize("fmt,g,M,N,K", [
    (pq.FMT_NVFP4, 16, 1000, 3001, 96), (pq.FMT_NVFP4, 16, 1000, 3001, 32), (pq.FMT_INT4, 64, 1000, 3001, 192),
    (pq.FMT_NVFP4, 16, 1000, 3001, 480), (pq.FMT_NVFP4, 16, 1000, 3001, 512), (pq.FMT_NVFP4, 16, 1000, 3001, 544), (pq.FMT_INT4, 64, 1000, 3001, 576),   # 128 x 192 tiles from K = 512 on
    (pq.FMT_NVFP4, 16, 65, 131, 32), (pq.FMT_INT4, 64, 65, 131, 64), (pq.FMT_NVFP4, 16, 129, 257, 160), (pq.FMT_INT3, 64, 130, 390, 448)])
def test_output_error_against_the_unquantized_product(fmt, g, M, N, K):
    """Both tiles of the unquantized product, ragged edges, one step of K and fewer than its stages, a last step of 32.  An
    element of either product is off by at most eps = (K + 4) 2^-24 sum |x||w|, so ||Y||^2 by 2 ||Y|| ||eps|| + ||eps||^2, and the
    error's numerator by the same with the difference in Y's place and 2 eps."""
    gen = torch.Generator(device=DEV).manual_seed(M + N + K + g)
    xs = [(torch.randn((M, K), generator=gen, device=DEV) * torch.exp(torch.randn(K, generator=gen, device=DEV))).to(torch.bfloat16) for _ in range(2)]
    w = torch.randn((N, K), generator=gen, device=DEV).to(torch.bfloat16)
    sa, sw = sum(x.double().square().sum(0) for x in xs), w.double().square().sum(0)
    Ta, Tw = ((t.float().abs().max() / 2688).reshape(1) for t in (torch.cat(xs), w))
    perm = torch.empty(K, dtype=torch.int32, device=DEV)
    rep = pq.pq_select_perm_output_error(fmt, g, sa, sw, xs, w, float(Ta), float(Tw), perm)
    x = torch.cat(xs)
    y = x.double() @ w.double().t()
    d = y - _dequantized(fmt, g, x, Ta)[2] @ _dequantized(fmt, g, w, Tw)[2].t()
    eps = 1.2 * (K + 4) * 2.0 ** -24 * (x.double().abs() @ w.double().abs().t()).norm()       # 1.2: quantized magnitudes are larger
    assert abs(rep.sum_x2 - y.norm() ** 2) <= 2 * y.norm() * eps + eps ** 2
    assert abs(rep.e_orig * rep.sum_x2 - d.norm() ** 2) <= 2 * d.norm() * 2 * eps + 4 * eps ** 2
