"""The work that users of the quantized layer step give this library, as cases that can be timed and compared.

Every case is one pass through the public entry points in the order in which a training or inference program calls
them, on buffers and a workspace that such a program keeps from step to step.  Five kinds:

  linear     one training step of a linear layer: both quantizers forward (index, soft value, marginal PMF, entropy),
             the forward product, both backward products, both quantizers backward
  conv       the same for a convolutional layer on [B, H, W, C] activations
  quantizer  forward and backward of the quantizer alone on a flat weight tensor
  entropy    the steps of entropy-constrained training on a weight tensor: marginal PMF, entropy and its gradient, the
             probabilistic draw, the Huffman-coded size
  infer      a linear layer at inference: indices of the activations, product with the stored weight indices

Fields: `bits` 2..8 (weights: 2^bits - 1 signed levels; activations: 2^bits unsigned levels after a ReLU, which for
eight bits are stored with an offset, or 2^bits - 1 signed ones where `act` is "outliers"); `kappa` the sharpness times
the squared step, or 0 for the initial sharpness 500 of training; `top` the truncation of the activations' PMF (0: none).
Step sizes follow the initialisation rule 2 mean|t| / sqrt(2^(bits - 1)).
"""
import math

import torch

import paper_2501_09849_amd as cdl

HALF = math.sqrt(2.0 / math.pi)      # mean |N(0, 1)|
ALPHA_0 = 500.0                      # sharpness at the start of training


def _linear(M, N, K, bits, act="relu", kappa=4.0, top=0, fused=False):
    return {"kind": "linear", "M": M, "N": N, "K": K, "bits": bits, "act": act, "kappa": kappa, "top": top, "fused": fused}


def _conv(B, H, W, C, N, R, stride, bits=4, kappa=4.0, top=0):
    return {"kind": "conv", "B": B, "H": H, "W": W, "C": C, "N": N, "R": R, "stride": stride, "bits": bits, "kappa": kappa, "top": top}


def _quantizer(n, bits, kappa):
    return {"kind": "quantizer", "n": n, "bits": bits, "kappa": kappa}


def _entropy(n, bits, kappa=4.0):
    return {"kind": "entropy", "n": n, "bits": bits, "kappa": kappa}


def _infer(M, N, K, bits, act="relu", fused=False):
    return {"kind": "infer", "M": M, "N": N, "K": K, "bits": bits, "act": act, "fused": fused}


def listed():
    return [
        # a toy layer: launches and host time
        dict(_linear(32, 128, 256, 4), name="linear_tiny"),
        # a thin layer in window-matrix form (first stage of a small CNN): long and narrow
        dict(_linear(131072, 16, 144, 4), name="linear_thin_windows"),
        # the last layer of an ImageNet CNN, kept at eight bits: ragged width, unsigned activations stored with an offset
        dict(_linear(256, 1000, 512, 8), name="linear_classifier_u8"),
        # a 3 x 3 layer of an ImageNet CNN in window-matrix form, backward products and quantizers in one call
        dict(_linear(50176, 256, 2304, 4, fused=True), name="linear_windows_fused"),
        # the up-projection of a transformer MLP at eight bits, activations with outliers: the largest step
        dict(_linear(65536, 3072, 768, 8, act="outliers"), name="linear_transformer_mlp"),
        # convolutional layers: the first stage of a small CNN, a middle stage and a stride-2 transition of an ImageNet CNN
        dict(_conv(128, 32, 32, 16, 16, 3, 1), name="conv_small_channels"),
        dict(_conv(256, 14, 14, 256, 256, 3, 1), name="conv_middle_stage"),
        dict(_conv(128, 56, 56, 64, 128, 3, 2), name="conv_stride2"),
        # all weights of a large CNN as one tensor, in mid-training and at the initial sharpness
        dict(_quantizer(25_600_000, 5, 4.0), name="quantizer_flat"),
        dict(_quantizer(25_600_000, 5, 0.0), name="quantizer_flat_initial"),
        # one weight matrix of a transformer MLP under the entropy constraint
        dict(_entropy(2_359_296, 8), name="entropy_weights"),
        # a few tokens through that layer
        dict(_infer(16, 3072, 768, 8, act="outliers"), name="infer_few_rows"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Sizes over the logarithm of the whole range, ragged ones as often as whole tiles; never beyond the largest listed case."""
    kind = rng.choice(["linear"] * 4 + ["conv"] * 3 + ["quantizer"] * 2 + ["entropy", "infer", "infer"])
    bits = rng.choice([2, 3, 4, 4, 6, 8, 8])
    kappa = rng.choice([4.0, 0.0, round(rng.uniform(3.0, 12.0), 2)])
    if kind in ("linear", "infer"):
        M = _log_int(rng, 32, 65536) if kind == "linear" else _log_int(rng, 1, 8192)
        N, K = _log_int(rng, 16, 3072), _log_int(rng, 64, 3072)
        if rng.random() < 0.5:      # widths of real layers are mostly multiples of 64
            N, K = (N + 63) // 64 * 64, (K + 63) // 64 * 64
        M = max(1, min(M, 65536 * 3072 * 768 // (N * K), 65536 * 1536 // max(N, K)))
        act = rng.choice(["relu", "outliers"])
        if kind == "infer":
            return _infer(M, N, K, bits, act, fused=K % 128 == 0 and (bits < 8 or act == "outliers") and rng.random() < 0.5)
        return _linear(M, N, K, bits, act, kappa, rng.choice([0, 0, 5]), fused=K % 4 == 0 and N > 32 and rng.random() < 0.4)
    if kind == "conv":
        H = rng.randint(7, 56)
        C, N = 16 * _log_int(rng, 1, 32), 4 * _log_int(rng, 4, 128)
        R, stride = rng.choice([1, 3, 3, 3, 5]), rng.choice([1, 1, 2])
        per_image = H * H * max(C, N, R * R * C * N // 512)
        B = max(1, min(_log_int(rng, 4, 256), 40_000_000 // per_image))
        return _conv(B, H, rng.choice([H, rng.randint(7, 56)]) if H * 56 * C * B < 40_000_000 else H, C, N, R, stride, bits, kappa,
                     rng.choice([0, 0, 5]))
    # the initial sharpness on wide level sets is left to the whole steps: there the step gradient is a sum that cancels to nothing
    if kind == "quantizer":
        n = _log_int(rng, 1000, 50_000_000)
        return _quantizer(n, bits, kappa) if kappa or bits <= 5 else _quantizer(n, rng.choice([4, 5]), kappa)
    return _entropy(_log_int(rng, 1000, 25_600_000), bits, kappa or 4.0)


# ---- quantizers -----------------------------------------------------------------------------------------------------

def _spec(lo, levels, step, kappa):
    """(lo, n_levels, step, sharpness)"""
    step = float(torch.tensor(step, dtype=torch.float32))
    return (lo, levels, step, kappa / (step * step) if kappa else ALPHA_0)


def _weight_spec(sigma, bits, kappa):
    half = 2 ** (bits - 1) - 1
    return _spec(-half, 2 * half + 1, 2.0 * sigma * HALF / math.sqrt(2.0 ** (bits - 1)), kappa)


def _act_spec(act, bits, kappa):
    if act == "outliers":
        half = 2 ** (bits - 1) - 1
        return _spec(-half, 2 * half + 1, 2.0 * (0.99 + 0.08) * HALF / math.sqrt(2.0 ** (bits - 1)), kappa)
    return _spec(0, 2 ** bits, 2.0 * HALF / math.sqrt(2.0 ** (bits - 1)), kappa)


def _flat_spec(bits, kappa):
    # weights N(0, 0.02^2) on 31 levels 0.004 apart, the same span for other level counts
    half = 2 ** (bits - 1) - 1
    return _spec(-half, 2 * half + 1, 0.06 / half, kappa)


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _activations(act, shape, gen):
    x = torch.randn(shape, device="cuda", generator=gen)
    if act == "outliers":     # one entry in a hundred is eight times as large
        m = torch.rand(shape, device="cuda", generator=gen) < 0.01
        return torch.where(m, x * 8.0, x)
    return x.abs_()


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _i8(*shape):
    return torch.empty(shape, dtype=torch.int8, device="cuda")


def _workspace(*sizes):
    return torch.empty(max(256, *sizes), dtype=torch.uint8, device="cuda")


def _side(theta, spec, top):
    """Buffers of one quantized tensor: indices, soft values, PMF, entropy, gradients."""
    return {"theta": theta, "n": theta.numel(), "spec": spec, "top": top, "idx": _i8(*theta.shape), "soft": _f32(*theta.shape),
            "marg": _f32(spec[1]), "H": _f32(1), "hat": _f32(*theta.shape), "d": _f32(*theta.shape), "d_step": _f32(1), "d_alpha": _f32(1),
            "off": cdl.cdl_index_offset(*spec)}


def _conv_geom(c):
    return (c["B"], c["H"], c["W"], c["C"], c["N"], c["R"], c["R"], c["stride"], c["R"] // 2)


def _conv_out(c):
    pad = c["R"] // 2
    return (c["H"] + 2 * pad - c["R"]) // c["stride"] + 1, (c["W"] + 2 * pad - c["R"]) // c["stride"] + 1


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = c["kind"]
    if kind in ("quantizer", "entropy"):
        n, spec = c["n"], _flat_spec(c["bits"], c["kappa"])
        w = _side(torch.randn(n, device="cuda", generator=gen) * 0.02, spec, 0)
        s = {"kind": kind, "w": w, "G": torch.randn(n, device="cuda", generator=gen)}
        if kind == "entropy":
            s.update(U=torch.rand(n, device="cuda", generator=gen), drawn=_i8(n), scale=0.01 * n,
                     counts=torch.empty(spec[1], dtype=torch.int64, device="cuda"), bits=torch.empty(1, dtype=torch.int64, device="cuda"),
                     rate=_f32(1), ws=_workspace(cdl.quantize_workspace_bytes(n, spec[1]), cdl.huffman_workspace_bytes(n)))
        else:
            s["ws"] = _workspace(cdl.quantize_workspace_bytes(n, spec[1]))
        return s
    if kind == "infer":
        M, N, K = c["M"], c["N"], c["K"]
        sigma = math.sqrt(2.0 / K)
        ws_, xs = _weight_spec(sigma, c["bits"], 4.0), _act_spec(c["act"], c["bits"], 4.0)
        X = _activations(c["act"], (M, K), gen)
        W = torch.randn((N, K), device="cuda", generator=gen) * sigma
        Wi = _i8(N, K)
        cdl.cdl_quantize_fwd(W, N * K, *ws_, Wi)      # a deployed layer keeps the indices only
        off = cdl.cdl_index_offset(*xs)
        return {"kind": kind, "X": X, "Wi": Wi, "xs": xs, "dw": ws_[2], "off": off, "MNK": (M, N, K), "fused": c["fused"], "Xi": _i8(M, K),
                "Y": _f32(M, N), "ws": _workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))}
    if kind == "linear":
        M, N, K = c["M"], c["N"], c["K"]
        sigma = 0.02 if c["act"] == "outliers" else math.sqrt(2.0 / K)
        x_shape, w_shape, y_shape, act = (M, K), (N, K), (M, N), c["act"]
        need = [cdl.qgemm_fwd_offset_workspace_bytes(M, N, K), cdl.qgemm_bwd_workspace_bytes(M, N, K)]
    else:
        B, H, W_, C, N, R, S, stride, pad = geom = _conv_geom(c)
        sigma = math.sqrt(2.0 / (R * S * C))
        x_shape, w_shape, y_shape, act = (B, H, W_, C), (N, R, S, C), (B,) + _conv_out(c) + (N,), "relu"
        need = None
    xs, wsp = _act_spec(act, c["bits"], c["kappa"]), _weight_spec(sigma, c["bits"], c["kappa"])
    x = _side(_activations(act, x_shape, gen), xs, c["top"])
    w = _side(torch.randn(w_shape, device="cuda", generator=gen) * sigma, wsp, 0)
    if need is None:
        need = [cdl.qconv_fwd_workspace_bytes(N, x["off"]), cdl.qconv_bwd_weights_workspace_bytes(*geom),
                cdl.qconv_bwd_activations_workspace_bytes(*geom)]
    s = {"kind": kind, "x": x, "w": w, "G": torch.randn(y_shape, device="cuda", generator=gen), "Y": _f32(*y_shape),
         "ws": _workspace(cdl.quantize_workspace_bytes(x["n"], xs[1]), cdl.quantize_workspace_bytes(w["n"], wsp[1]), *need)}
    if kind == "linear":
        s.update(MNK=(M, N, K), fused=c["fused"])
    else:
        s["geom"] = geom
    return s


# ---- one pass -------------------------------------------------------------------------------------------------------

def _forward(t, ws):
    cdl.cdl_quantize_fwd(t["theta"], t["n"], *t["spec"], t["idx"], t["soft"], t["marg"], t["H"], ws, top_k=t["top"])


def _backward(t, ws):
    cdl.cdl_quantize_bwd(t["theta"], t["hat"], t["n"], *t["spec"], t["d"], t["d_step"], t["d_alpha"], ws, top_k=t["top"])


def _outputs(t):
    return [t["idx"], t["soft"], t["marg"], t["H"], t["d"], t["d_step"], t["d_alpha"]]


def run(state):
    s = state
    kind, ws = s["kind"], s["ws"]
    if kind == "linear":
        x, w, Y, G = s["x"], s["w"], s["Y"], s["G"]
        M, N, K = s["MNK"]
        dx, dw = x["spec"][2], w["spec"][2]
        _forward(w, ws)
        _forward(x, ws)
        if x["off"]:
            cdl.cdl_qgemm_fwd_offset(x["idx"], w["idx"], M, N, K, dx, dw, x["off"], 0, None, Y, ws)
        else:
            cdl.cdl_qgemm_fwd(x["idx"], w["idx"], M, N, K, dx, dw, None, Y, ws)
        if s["fused"]:
            cdl.cdl_qgemm_bwd_quantize_bwd(G, x["idx"], w["idx"], M, N, K, x["theta"], *x["spec"], dw, x["d"], x["d_step"], x["d_alpha"], None, ws,
                                           top_k=x["top"], theta_b=w["theta"], qparams_b=w["spec"], d_theta_b=w["d"], d_delta_b=w["d_step"],
                                           d_alpha_b=w["d_alpha"])
        else:
            if x["off"]:
                cdl.cdl_qgemm_bwd_offset(G, x["idx"], w["idx"], M, N, K, dx, dw, x["off"], 0, x["hat"], w["hat"], ws)
            else:
                cdl.cdl_qgemm_bwd(G, x["idx"], w["idx"], M, N, K, dx, dw, x["hat"], w["hat"], ws)
            _backward(x, ws)
            _backward(w, ws)
        return [Y] + _outputs(x) + _outputs(w)
    if kind == "conv":
        x, w, Y, G, geom = s["x"], s["w"], s["Y"], s["G"], s["geom"]
        dx, dw = x["spec"][2], w["spec"][2]
        _forward(w, ws)
        _forward(x, ws)
        cdl.cdl_qconv_fwd(x["idx"], w["idx"], *geom, dx, dw, None, Y, ws, x_offset=x["off"])
        cdl.cdl_qconv_bwd_weights(G, x["idx"], *geom, dx, w["hat"], ws, x_offset=x["off"])
        cdl.cdl_qconv_bwd_activations(G, w["idx"], *geom, dw, x["hat"], ws)
        _backward(x, ws)
        _backward(w, ws)
        return [Y] + _outputs(x) + _outputs(w)
    if kind == "quantizer":
        w = s["w"]
        _forward(w, ws)
        cdl.cdl_quantize_bwd(w["theta"], s["G"], w["n"], *w["spec"], w["d"], w["d_step"], w["d_alpha"], ws)
        return _outputs(w)
    if kind == "entropy":
        w = s["w"]
        n, spec = w["n"], w["spec"]
        cdl.cdl_quantize_draw(w["theta"], s["U"], n, *spec, s["drawn"])
        cdl.cdl_quantize_fwd(w["theta"], n, *spec, w["idx"], None, w["marg"], w["H"], ws)
        cdl.cdl_entropy_bwd(w["theta"], w["marg"], n, *spec, s["scale"], s["G"], w["d"], w["d_step"], w["d_alpha"], ws)
        cdl.cdl_huffman_bits(w["idx"], n, spec[0], spec[1], s["counts"], s["bits"], s["rate"], ws)
        return [s["drawn"], w["idx"], w["marg"], w["H"], w["d"], w["d_step"], w["d_alpha"], s["counts"], s["bits"], s["rate"]]
    X, Y, xs = s["X"], s["Y"], s["xs"]
    M, N, K = s["MNK"]
    if s["fused"]:
        cdl.cdl_qgemm_fwd_quantize(X, *xs, s["Wi"], M, N, K, s["dw"], Y)
        return [Y]
    cdl.cdl_quantize_fwd(X, M * K, *xs, s["Xi"])
    if s["off"]:
        cdl.cdl_qgemm_fwd_offset(s["Xi"], s["Wi"], M, N, K, xs[2], s["dw"], s["off"], 0, None, Y, ws)
    else:
        cdl.cdl_qgemm_fwd(s["Xi"], s["Wi"], M, N, K, xs[2], s["dw"], None, Y, ws)
    return [Y, s["Xi"]]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    """Bytes: inputs read once, returned outputs written once.  Operations: the three products (two per multiply-add)."""
    c = case
    if c["kind"] == "quantizer":
        return {"bytes": 17 * c["n"], "flops": 0}                # theta, g; index, soft value, gradient
    if c["kind"] == "entropy":
        return {"bytes": 18 * c["n"], "flops": 0}                # theta, u, g; two indices, gradient
    if c["kind"] == "infer":
        M, N, K = c["M"], c["N"], c["K"]
        return {"bytes": 4 * M * K + N * K + 4 * M * N + (0 if c["fused"] else M * K), "flops": 2 * M * N * K}
    if c["kind"] == "linear":
        nx, nw, ny = c["M"] * c["K"], c["N"] * c["K"], c["M"] * c["N"]
        macs = c["M"] * c["N"] * c["K"]
    else:
        P, Q = _conv_out(c)
        nx, nw, ny = c["B"] * c["H"] * c["W"] * c["C"], c["N"] * c["R"] * c["R"] * c["C"], c["B"] * P * Q * c["N"]
        macs = ny * c["R"] * c["R"] * c["C"]
    return {"bytes": 13 * (nx + nw) + 8 * ny, "flops": 6 * macs}  # theta; index, soft value, gradient; g and y


def tolerance(case):
    """32-bit results.  The scalar gradients are sums over signed terms, so that rounding shows multiplied by how far they cancel,
    further at the initial sharpness, where the soft value hardly depends on the step.  Indices: ties; draws: numbers next to a boundary."""
    if case["kind"] == "infer":
        return {"rel": 1e-6, "differ": 1e-6}
    if case["kind"] == "entropy":
        return {"rel": 5e-5, "max": 1e-3, "differ": 1e-5}
    return {"rel": 5e-5 if case["kappa"] else 2e-4, "max": 1e-3, "differ": 1e-6}
