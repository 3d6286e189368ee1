"""GPU parity of the up projection for every width and code size the tuned kernels do not take: fp32 precision, edges of the
channel blocks, the smallest and the largest width, large activations."""
import numpy as np
import pytest
import torch

import floe_synth as S
import oracle as O

pytestmark = pytest.mark.gpu

# products of fp16 activations and integer codes are exact in fp32; a unit of 64 codes is four chains of 16 roundings, its
# group terms and the d / 64 units of a channel add at most 30 more: each 2^-24 of partial sums a few times rms(v)
BAR = 2e-6


@pytest.mark.parametrize("d,f,bits,group,T,scale", [
    (512, 1, 2, 64, 1, 1.0), (512, 63, 4, 32, 2, 1.0), (1536, 64, 3, 64, 1, 1.0), (2560, 65, 4, 128, 3, 1.0),
    (8192, 129, 2, 256, 1, 1.0), (8192, 7, 8, 64, 1, 1.0), (5120, 130, 1, 32, 2, 1.0), (1024, 33, 8, 128, 2, 1.0),
    (3072, 40, 3, 32, 1, 1.0), (2560, 30, 2, 64, 2, 3000.0), (1536, 20, 1, 64, 1, 8000.0), (4096, 30, 8, 64, 1, 8000.0),
])
def test_up_gemv_of_untuned_shapes(d, f, bits, group, T, scale):
    import gpu_common as G
    import paper_2505_05950_amd as F
    w_up, gd = S.expert_weights(95, 3, d, f)
    ex_np, ex_dev = G.make_expert(w_up, gd, bits, group)
    x = (S.tokens(95, 3, T, d).astype(np.float32) * scale).astype(np.float16)
    assert np.isfinite(x).all()
    v = F.floe_up_gemv(ex_dev.up_codes, ex_dev.up_scale, ex_dev.up_zero, G.dev(x), d, bits, group)
    torch.cuda.synchronize()
    v = v.cpu().numpy().astype(np.float64)
    wd = O.dequantize(*ex_np[:3], d, bits, group).astype(np.float64)
    for t in range(T):
        ref = O.up_gemv(*ex_np[:3], d, bits, group, x[t]).astype(np.float64)
        # the size of what cancels: one rounding of a partial sum is measured against it
        size = np.sqrt(np.mean(wd ** 2 @ x[t].astype(np.float64) ** 2))
        assert np.abs(v[t] - ref).max() <= BAR * size, (t, np.abs(v[t] - ref).max() / size)


@pytest.mark.parametrize("d,f,bits,group,T,scale", [
    (1536, 200, 2, 64, 1, 1.0), (2560, 333, 4, 128, 3, 1.0), (3072, 130, 3, 64, 16, 1.0), (1536, 70, 4, 32, 2, 1.0),
    (2560, 77, 2, 256, 1, 1.0), (3072, 40, 3, 32, 2, 1.0), (1536, 1500, 3, 128, 8, 1.0),
    (2560, 130, 2, 64, 2, 3000.0), (3072, 150, 4, 64, 1, 8000.0), (1536, 160, 3, 32, 1, 1e-5), (2560, 170, 4, 128, 2, 1e-5),
    (3072, 3000, 3, 64, 40, 1.0),  # more than one kernel takes, too few for the matrix cores, whose INT3 is good to 1e-5
])
def test_v_inside_a_one_expert_call_at_widths_between_the_powers_of_two(d, f, bits, group, T, scale):
    """The same bar for the v that a small call forms on its way to y: gate columns whose sum is 32 (SiLU leaves it as it is) and
    down rows with a single one make y = 32 v, exactly."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    w_up, _ = S.expert_weights(96, 3, d, f)
    gd = np.zeros((f, 2, d), np.float16)
    x0 = np.float16(2.0 ** int(np.log2(scale)))  # (as large as the other activations: subnormal in the smallest case)
    gd[:, 0, :64] = np.float16(0.5 / x0)
    gd[np.arange(f), 1, np.arange(f)] = 1.0
    ex_np, ex_dev = G.make_expert(w_up, gd, bits, group)
    x = (S.tokens(96, 3, T, d).astype(np.float32) * scale).astype(np.float16)
    x[:, :64] = x0
    tau = np.full((T,), -1.0, np.float32)  # every channel
    y, idx, count = F.floe_expert_ffn_sparse(ex_dev, G.dev(x), G.dev(tau), None, torch.zeros((T, d), device=G.DEV))
    torch.cuda.synchronize()
    y, idx, count = y.cpu().numpy().astype(np.float64), idx.cpu().numpy(), count.cpu().numpy()
    assert (count == f).all() and (idx == np.arange(f)).all() and not y[:, f:].any()
    wd = O.dequantize(*ex_np[:3], d, bits, group).astype(np.float64)
    for t in range(T):
        ref = O.up_gemv(*ex_np[:3], d, bits, group, x[t]).astype(np.float64)
        size = np.sqrt(np.mean(wd ** 2 @ x[t].astype(np.float64) ** 2))
        err = np.abs(y[t, :f] / 32.0 - ref).max() / size
        assert err <= BAR, (t, err)
