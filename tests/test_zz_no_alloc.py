"""The entry point that allocates nothing, moeca_forward_noalloc, against
the existing entry point it is a variant of: moeca_step on an uncached
(MOECA_MODE_FULL) layer, which runs the same kernels on a caller-bound
workspace.  Two calls in a row through the C ABI, the second on a smaller
input (fewer samples), each compared with moeca_step's output for the same
samples (max relative error 2e-2 in bf16, 1e-4 in fp32; the kernels are the
same, so the outputs are expected to be bit-identical and the test reports
whether they are).  Also: sizes beyond the library's scratch array and
sample counts outside [1, B] are refused with an error.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2606_15615_amd import _lib
from paper_2606_15615_amd.layer import MoecaLayer, device_to_np, np_to_device
from paper_2606_15615_amd.synth import LayerShape, Synth, WORKLOADS

TOL = {"bf16": 2e-2, "fp32": 1e-4}


def say(msg):
    print(msg, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _lib.load()


def _widen(a, dtype):
    if dtype == "bf16":
        return (np.asarray(a, np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    return np.asarray(a, np.float32).astype(np.float64)


def _rel_err(a, b, dtype):
    a64, b64 = _widen(a, dtype), _widen(b, dtype)
    den = np.abs(b64).max()
    return float(np.abs(a64 - b64).max() / den) if den > 0 else float(np.abs(a64).max())


CASES = [
    # the benchmarked layer's widths (d=1152, 16 experts, top-2, 4608 hidden)
    # at 2 of its 8 samples of 1024 tokens, then 1
    (LayerShape(d=1152, E=16, k=2, d_ff=4608, B=8, N=1024, dtype="bf16"), "gelu_tanh", 2, 1),
    # 256 tokens x 4 samples, then 3 (ragged last tiles)
    (LayerShape(d=1152, E=16, k=2, d_ff=4608, B=4, N=256, dtype="bf16"), "gelu_tanh", 4, 3),
    # gated experts with a shared expert, ragged token count
    (LayerShape(d=256, E=8, k=2, d_ff=128, B=3, N=77, dtype="bf16", ffn="swiglu", n_shared=1),
     "swiglu", 3, 1),
    # 32 rows per expert, then 16: the weight-streaming tiles, K in four pieces
    (LayerShape(d=576, E=16, k=2, d_ff=2304, B=2, N=128, dtype="bf16"), "gelu_erf", 2, 1),
    # fp32 layer with erf GELU
    (LayerShape(d=384, E=8, k=2, d_ff=1536, B=2, N=256, dtype="fp32"), "gelu_erf", 2, 1),
]


@pytest.mark.parametrize("shape,act,first,second", CASES)
def test_noalloc_matches_step(shape, act, first, second):
    import torch
    say(f"  no-alloc forward: {shape} act={act}, calls with {first} then {second} samples")
    sy = Synth(shape, 40)
    W_r, b_r, W_up, W_down = sy.weights()
    L = MoecaLayer(shape.d, shape.E, shape.k, shape.d_ff, batch=shape.B, tokens=shape.N,
                   mode=_lib.MOECA_MODE_FULL, dtype=shape.dtype, act=act,
                   n_shared=shape.n_shared)
    dev = L.device
    L.set_weights(np_to_device(W_r, dev), None, np_to_device(W_up, dev),
                  np_to_device(W_down, dev))
    if shape.n_shared:
        L.set_shared(*[np_to_device(w, dev) for w in sy.shared_weights()])
    act_np = np.uint16 if shape.dtype == "bf16" else np.float32
    x = np_to_device(next(sy.trajectory(1)), dev)
    ref = torch.zeros_like(x)
    L.reset()
    L.step(x, 0, ref)
    torch.cuda.synchronize()
    ref_np = device_to_np(ref, act_np)
    stream = torch.cuda.current_stream(dev).cuda_stream
    for samples in (first, second):
        xs = x[:samples].contiguous()
        out = torch.full_like(xs, -1)      # poisoned: every element must be written
        _lib.moeca_forward_noalloc(L.h, xs.data_ptr(), samples, out.data_ptr(), stream)
        torch.cuda.synchronize()
        got = device_to_np(out, act_np)
        want = ref_np[:samples]
        e = _rel_err(got, want, shape.dtype)
        say(f"    {samples} samples: max rel err {e:.3g}, bit-identical {np.array_equal(got, want)}")
        assert e <= TOL[shape.dtype]
    L.close()


def test_noalloc_rejects_what_it_cannot_hold():
    import torch
    p = _lib.moeca_policy_default()
    p.mode, p.batch, p.tokens = _lib.MOECA_MODE_FULL, 8, 1024
    h = _lib.moeca_layer_create(1152, 16, 2, 4608, p)     # the full benchmarked batch
    x = torch.zeros((8, 1024, 1152), dtype=torch.int16, device="cuda:0")
    out = torch.zeros_like(x)
    stream = torch.cuda.current_stream().cuda_stream
    try:
        with pytest.raises(_lib.MoecaError, match="bytes of scratch"):
            _lib.moeca_forward_noalloc(h, x.data_ptr(), 8, out.data_ptr(), stream)
        with pytest.raises(_lib.MoecaError, match="samples must be in"):
            _lib.moeca_forward_noalloc(h, x.data_ptr(), 9, out.data_ptr(), stream)
        with pytest.raises(_lib.MoecaError, match="samples must be in"):
            _lib.moeca_forward_noalloc(h, x.data_ptr(), 0, out.data_ptr(), stream)
        with pytest.raises(_lib.MoecaError, match="weights are not bound"):
            _lib.moeca_forward_noalloc(h, x.data_ptr(), 1, out.data_ptr(), stream)
    finally:
        _lib.moeca_layer_destroy(h)
    torch.cuda.synchronize()
    assert int(out.abs().sum()) == 0      # nothing ran
