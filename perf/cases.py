"""The work this library does for its users, as cases that can be timed and compared.

Every path is one kind of program: decoding token by token, prefill with a carried state, inference over whole
sequences, and the training steps of the attention (bf16 and fp32), of the gated layer, of the non-causal classifier
and of the short-long convolution.  `listed()` holds fixed sizes (the named workloads of the package and of bench.py,
or ragged ones near them), `draw()` more of the same ranges.
"""
import math

import torch

from paper_2406_08128_amd import binding

EPS = 1e-5          # of the normalisation in the gated paths (any small constant; the value does not change the work)


def listed():
    return [
        # One token of one sequence, 12 heads: the smallest call, nothing but latency and launches.
        {"name": "decode_one", "path": "decode", "B": 1, "H": 12, "dk": 64, "dv": 64},
        # A serving batch decoding together (bench.py's --mode decode): the fp32 states are read and written once.
        {"name": "decode_batch", "path": "decode", "B": 256, "H": 12, "dk": 64, "dv": 64},
        # A few prompts of an odd length, continued from a carried state and handing the next one on.
        {"name": "prefill_ragged", "path": "prefill", "B": 3, "H": 12, "N": 1531, "dk": 64, "dv": 64},
        # Inference over a full batch of 4K sequences (the LRA-shaped workload).
        {"name": "lra_fwd", "path": "fwd", "B": 32, "H": 8, "N": 4096, "dk": 64, "dv": 64, "dtype": "bf16"},
        # The longest sequences with the widest heads, positive feature map (the long-sequence workload).
        {"name": "long_fwd", "path": "fwd", "B": 1, "H": 16, "N": 65536, "dk": 128, "dv": 128, "dtype": "bf16"},
        # Forward + backward at the language-model shape: the headline workload.
        {"name": "lm_train", "path": "train", "B": 4, "H": 12, "N": 16384, "dk": 64, "dv": 64, "dtype": "bf16"},
        # Forward + backward with a rectangular state (the mixed-head workload).
        {"name": "mixed_train", "path": "train", "B": 8, "H": 12, "N": 4096, "dk": 64, "dv": 128, "dtype": "bf16"},
        # The fp32 accuracy path, forward + backward, an odd length.
        {"name": "f32_train", "path": "train", "B": 2, "H": 12, "N": 3001, "dk": 64, "dv": 64, "dtype": "f32"},
        # One training step of the gated layer's token mixing (Z, V, G -> Y and all gradients) at an ordinary context.
        {"name": "layer_train", "path": "layer", "B": 4, "H": 12, "N": 2048, "dk": 64, "dv": 64},
        # One training step of the unmasked, gated classifier on a batch padded to its own longest sequence.
        {"name": "noncausal_train", "path": "noncausal", "B": 32, "H": 8, "N": 3517, "dk": 64, "dv": 64},
        # One training step of the short-long convolution at the LRA-shaped width; the kernel's weights change with
        # every step, so its spectrum is part of the step.
        {"name": "conv_train_lra", "path": "conv", "B": 32, "d": 512, "L": 4096, "m": 9, "dtype": "bf16"},
        # The same at the language-model width and length: the largest case.
        {"name": "conv_train_lm", "path": "conv", "B": 4, "d": 768, "L": 16384, "m": 9, "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _heads(rng):
    return rng.choice([(64, 64), (64, 64), (64, 128), (128, 64), (128, 128)])


def draw(rng):
    """One more case of the listed paths.  Lengths are spread over their logarithm and mostly odd; the batch is then
    limited so that no case moves more than the listed ones of its path."""
    path = rng.choice(["decode", "prefill", "fwd", "train", "train", "layer", "noncausal", "conv"])
    H = rng.choice([4, 8, 12, 16])
    dk, dv = _heads(rng)
    if path == "decode":
        B = _log_int(rng, 1, 256)
        return {"path": path, "B": min(B, max(1, 256 * 12 * 4096 // (H * dk * dv))), "H": H, "dk": dk, "dv": dv}
    if path == "conv":
        L = _log_int(rng, 200, 16384)
        if rng.random() < 0.5:
            L = max(8, L // 8 * 8)
        d = rng.choice([128, 256, 512, 768])
        B = _log_int(rng, 1, 32)
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        most = 4 * 768 * 16384 // (2 if dtype == "f32" else 1)
        return {"path": path, "B": min(B, max(1, most // (d * L))), "d": d, "L": L, "m": rng.randint(3, 12),
                "dtype": dtype}
    case = {"path": path, "B": _log_int(rng, 1, 32), "H": H, "N": 0, "dk": dk, "dv": dv}
    most = 4 * 12 * 16384 * 128                 # elements of B*H*N*(dk+dv) at the language-model shape
    if path == "prefill":
        case["N"], most = _log_int(rng, 16, 16384), most // 4
    elif path == "fwd":
        case["N"], case["dtype"] = _log_int(rng, 512, 65536), "bf16"
        most = 16 * 65536 * 256                 # the long-sequence workload
    elif path == "train":
        case["dtype"] = "f32" if rng.random() < 0.33 else "bf16"
        case["N"] = _log_int(rng, 256, 16384)
        most = most // 4 if case["dtype"] == "f32" else most
    else:
        case["N"] = _log_int(rng, 256, 8192)
    case["B"] = min(case["B"], max(1, most // (H * case["N"] * (dk + dv))))
    return case


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def randn(*shape):
        return torch.randn(*shape, generator=g, dtype=torch.float32, device="cuda")

    path = case["path"]
    bf = torch.bfloat16
    if path == "conv":
        B, d, L, m = case["B"], case["d"], case["L"], case["m"]
        dt = bf if case["dtype"] == "bf16" else torch.float32
        t = torch.arange(L, dtype=torch.float32, device="cuda")
        return {"path": path, "X": randn(B, d, L).to(dt), "dZ": randn(B, d, L).to(dt),
                "w_short": (randn(d, m) / m).contiguous(),
                # a decaying kernel as long as the sequence, of unit energy
                "k_long": (randn(d, L) * torch.exp(-4.0 * t / L)[None, :] * (8.0 / L) ** 0.5).contiguous()}
    B, H, dk, dv = case["B"], case["H"], case["dk"], case["dv"]
    silu = torch.nn.functional.silu
    if path == "decode":
        # a state some hundred tokens have gone into
        return {"path": path, "q": (randn(B, H, dk) / 8).to(bf), "k": (randn(B, H, dk) / 8).to(bf),
                "v": randn(B, H, dv).to(bf), "g": silu(randn(B, H, dv)).to(bf), "S": randn(B, H, dk, dv).contiguous()}
    N = case["N"]
    dt = torch.float32 if case.get("dtype") == "f32" else bf
    s = {"path": path, "V": randn(B, H, N, dv).to(dt)}
    if path == "layer":
        n = randn(4, H, dk)
        s["Z"] = randn(B, H, N, dk).to(bf)
        # learnable scales and offsets around the 1/8 spread of the plain queries and keys
        s["affine"] = torch.stack([(1 + n[0] / 4) / 8, n[1] / 32, (1 + n[2] / 4) / 8, n[3] / 32]).contiguous()
    elif path == "fwd" and dk == 128 and dv == 128:
        # the positive feature map of the long-sequence workload: the state grows with the position
        elu = torch.nn.functional.elu
        s["Q"] = ((elu(randn(B, H, N, dk)) + 1) / 128).to(dt)
        s["K"] = ((elu(randn(B, H, N, dk)) + 1) / 128).to(dt)
    else:
        s["Q"] = (randn(B, H, N, dk) / 8).to(dt)
        s["K"] = (randn(B, H, N, dk) / 8).to(dt)
    if path == "prefill":
        s["S_in"] = randn(B, H, dk, dv).contiguous()
    if path in ("layer", "noncausal"):
        s["G"] = silu(randn(B, H, N, dv)).to(bf)
        s["dY"] = randn(B, H, N, dv).to(bf)
    if path == "train":
        s["dO"] = randn(B, H, N, dv).to(dt)
    return s


def run(s):
    path = s["path"]
    if path == "decode":
        return {"y": binding.chela_linattn_step_gated(s["q"], s["k"], s["v"], s["g"], s["S"], EPS), "S": s["S"]}
    if path == "prefill":
        O, S_out = binding.chela_linattn_fwd_state(s["Q"], s["K"], s["V"], S_in=s["S_in"])
        return {"O": O, "S_out": S_out}
    if path == "fwd":
        return {"O": binding.chela_linattn_fwd(s["Q"], s["K"], s["V"])}
    if path == "train":
        O = binding.chela_linattn_fwd(s["Q"], s["K"], s["V"])
        dQ, dK, dV = binding.chela_linattn_bwd(s["Q"], s["K"], s["V"], s["dO"])
        return {"O": O, "dQ": dQ, "dK": dK, "dV": dV}
    if path == "layer":
        Y, O, saved = binding.chela_linattn_zfwd_gated(s["Z"], s["affine"], s["V"], s["G"], EPS, want_O=True,
                                                       want_saved=True)
        dO, dG = binding.chela_gate_norm_bwd(O, s["G"], s["dY"], EPS)
        dZ, d_affine, dV = binding.chela_linattn_zbwd_saved(s["Z"], s["affine"], s["V"], dO, saved)
        return {"Y": Y, "dG": dG, "dZ": dZ, "d_affine": d_affine, "dV": dV}
    if path == "noncausal":
        Y, O = binding.chela_linattn_noncausal_fwd_gated(s["Q"], s["K"], s["V"], s["G"], EPS, want_O=True)
        dO, dG = binding.chela_gate_norm_bwd(O, s["G"], s["dY"], EPS)
        dQ, dK, dV = binding.chela_linattn_noncausal_bwd(s["Q"], s["K"], s["V"], dO)
        return {"Y": Y, "dG": dG, "dQ": dQ, "dK": dK, "dV": dV}
    if path == "conv":
        spectrum = binding.chela_longconv_spectrum(s["k_long"])
        Z = binding.chela_shortlong_conv_fwd(s["X"], s["w_short"], spectrum)
        dX, dw, dk = binding.chela_shortlong_conv_bwd(s["X"], s["w_short"], spectrum, s["dZ"])
        return {"Z": Z, "dX": dX, "d_w_short": dw, "d_k_long": dk}
    raise ValueError(path)


def work(case):
    path = case["path"]
    es = 4 if case.get("dtype") == "f32" else 2
    if path == "conv":
        B, d, L, m = case["B"], case["d"], case["L"], case["m"]
        fft = 5.0 * L * math.log2(max(L, 2))            # 2 L real values, zero-padded, as L complex ones
        transforms = 5 * B * d + 2 * d                   # input, output, dZ, dv, v again; the kernel's and its gradient's
        return {"bytes": B * d * L * es * 4 + d * L * 8 + d * m * 8,
                "flops": transforms * fft + B * d * L * (4 * 6 + 3 * 2 * m)}
    B, H, dk, dv = case["B"], case["H"], case["dk"], case["dv"]
    if path == "decode":
        return {"bytes": B * H * (dk * dv * 8 + 4 * dk + 6 * dv), "flops": 4.0 * B * H * dk * dv}
    th = B * H * case["N"]
    fwd, bwd = 4.0 * th * dk * dv, 10.0 * th * dk * dv   # the recurrent form: state update and query; 5 such products
    if path == "prefill":
        return {"bytes": th * (2 * dk + 2 * dv) * 2 + B * H * dk * dv * 8, "flops": fwd}
    if path == "fwd":
        return {"bytes": th * (2 * dk + 2 * dv) * es, "flops": fwd}
    if path == "train":
        return {"bytes": th * (4 * dk + 4 * dv) * es, "flops": fwd + bwd}        # Q K V dO; O dQ dK dV
    if path == "layer":
        return {"bytes": th * (2 * dk + 6 * dv) * 2 + 32 * H * dk, "flops": fwd + bwd}   # Z V G dY; Y dG dZ dV
    return {"bytes": th * (4 * dk + 6 * dv) * 2, "flops": fwd + bwd}             # Q K V G dY; Y dG dQ dK dV


def tolerance(case):
    # About four times what was measured.  bf16: the calls differ from the fp64 oracle by 2.4e-3 (their outputs' own
    # rounding and that of the matrix cores' operands) and from themselves with the sums cut up differently (other
    # chunk and segment lengths, for the convolution the vector-ALU transforms) by 1e-4 to 1.5e-3, single values by
    # up to 0.02.  fp32: 5e-7 and 4e-6 for the attention, 1e-6 for the convolution.
    if case.get("dtype") == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}
