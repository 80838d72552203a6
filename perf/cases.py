"""The work that a user of this library has it do, as measurable cases.

Every case is one pass through the public entry points (``vx.gemm``,
``vx.vx_gemm``, ``vx.bmm``, ``vx.conv2d``) on operands that are in GPU memory
before the call.  The families, their sizes and their value distributions are
those of ``paper_2409_01075_amd/inputs.py`` and of the benchmark:

* ``sweep``      fp16 (M x 768) x (768 x 768), dynamic M = 1..512: the smallest
                 calls, where launches and latency count
* ``llm``        the three bf16 weight products of a decoder layer (4096, 11008),
                 M tokens from a single one (decode) to 8192 (prefill)
* ``encoder``    the four bf16 weight products of an encoder layer (768, 3072),
                 16 sequences of L tokens
* ``attention``  the two bf16 batched products of attention, scores Q K^T and
                 P V, 192 heads of 64, any length L (rows off 16-byte alignment
                 where L is not a multiple of 8)
* ``conv``       one fp16 NHWC convolution layer of a CNN: odd first layers over
                 three channels, 1x1, 3x3, 5x5, strides, any channel count
* ``gemm``       a plain product of any of the three types and any size

``exact`` is the same result in binary64 from plain torch.
"""
import math

import torch

from paper_2409_01075_amd import vx

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ABI_CODES = {"f32": vx.VX_F32, "f16": vx.VX_F16, "bf16": vx.VX_BF16}
ENCODER = [(768, 2304), (768, 768), (768, 3072), (3072, 768)]   # (K, N): QKV, output, FFN up, FFN down
LLM = [(4096, 4096), (4096, 11008), (11008, 4096)]              # (K, N): attention output, FFN up, FFN down
HEADS, HEAD_DIM = 16 * 12, 64


def listed():
    return [
        # a few rows of a dynamic-M stream, through the torch helper
        {"name": "sweep_f16_m37", "family": "sweep", "dtype": "f16", "m": 37, "entry": "gemm"},
        # a fuller call of the same stream, by pointers as an engine with its own buffers makes it
        {"name": "sweep_f16_m389", "family": "sweep", "dtype": "f16", "m": 389, "entry": "abi"},
        # decode: one token for each of seven requests
        {"name": "llm_bf16_m7", "family": "llm", "dtype": "bf16", "m": 7},
        # a short prompt (or a chunk of prefill beside decode)
        {"name": "llm_bf16_m279", "family": "llm", "dtype": "bf16", "m": 279},
        # a long prefill, the largest call
        {"name": "llm_bf16_m8192", "family": "llm", "dtype": "bf16", "m": 8192},
        # an encoder layer over a batch of 16 sequences of ragged length
        {"name": "encoder_bf16_l317", "family": "encoder", "dtype": "bf16", "l": 317},
        # attention at a length that leaves every row off 16-byte alignment
        {"name": "attention_bf16_l485", "family": "attention", "dtype": "bf16", "l": 485},
        # attention at a long aligned length
        {"name": "attention_bf16_l968", "family": "attention", "dtype": "bf16", "l": 968},
        # the workhorse layer of a CNN
        {"name": "conv_f16_3x3_c128", "family": "conv", "dtype": "f16", "n": 16, "hw": 56, "cin": 128, "cout": 128,
         "f": 3, "stride": 1, "pad": 1},
        # the first layer of a CNN: three channels, a large map
        {"name": "conv_f16_7x7_stem", "family": "conv", "dtype": "f16", "n": 16, "hw": 224, "cin": 3, "cout": 64,
         "f": 7, "stride": 2, "pad": 3},
        # single precision, ragged rows
        {"name": "gemm_f32_1021x3072x768", "family": "gemm", "dtype": "f32", "m": 1021, "n": 3072, "k": 768},
        # half precision with every size odd
        {"name": "gemm_f16_777x1111x533", "family": "gemm", "dtype": "f16", "m": 777, "n": 1111, "k": 533},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["sweep", "llm", "encoder", "attention", "conv", "conv", "gemm", "gemm"])
    if family == "sweep":
        return {"family": family, "dtype": "f16", "m": rng.randint(1, 512), "entry": rng.choice(["gemm", "abi"])}
    if family == "llm":
        return {"family": family, "dtype": "bf16", "m": _log_int(rng, 1, 8192)}
    if family == "encoder":
        return {"family": family, "dtype": "bf16", "l": rng.randint(1, 512)}
    if family == "attention":
        return {"family": family, "dtype": "bf16", "l": rng.randint(1, 1024)}
    if family == "conv":
        f = rng.choice([1, 1, 1, 3, 3, 3, 3, 5, 7, 11])
        stem = f >= 7
        cin = 3 if stem else rng.choice([8 * _log_int(rng, 2, 104), _log_int(rng, 3, 832)])
        case = {"family": family, "dtype": "f16", "n": _log_int(rng, 1, 64), "hw": _log_int(rng, 7, 384), "cin": cin,
                "cout": 16 * _log_int(rng, 1, 32), "f": f,
                "stride": (4 if f == 11 else 2) if stem or rng.random() < 0.25 else 1, "pad": f // 2}
        while True:    # at most 2^25 elements in or out and 1e11 operations: halve the batch, then the map
            o = _out_dim(case)
            if (max(case["hw"] ** 2 * cin, o * o * case["cout"]) * case["n"] <= 2 ** 25
                    and 2.0 * case["n"] * o * o * case["cout"] * f * f * cin <= 1e11):
                return case
            if case["n"] > 1:
                case["n"] //= 2
            else:
                case["hw"] = max(case["hw"] // 2, 7)
    case = {"family": "gemm", "dtype": rng.choice(["f32", "f32", "f16", "bf16"])}
    while True:
        case["m"], case["n"], case["k"] = (_log_int(rng, 16, 4096) for _ in range(3))
        if rng.random() < 0.5:    # half of them with rows that start on 16-byte boundaries
            case["n"], case["k"] = -(-case["n"] // 8) * 8, -(-case["k"] // 8) * 8
        if 2.0 * case["m"] * case["n"] * case["k"] <= 3e10:
            return case


def _out_dim(c):
    return (c["hw"] + 2 * c["pad"] - c["f"]) // c["stride"] + 1


def _products(c):
    """The (batch, M, N, K, std of B, kind of A) of each product of a GEMM case."""
    fam = c["family"]
    if fam == "sweep":
        return [(1, c["m"], 768, 768, None, "uniform")]
    if fam == "llm":
        return [(1, c["m"], n, k, 0.02, "normal") for k, n in LLM]
    if fam == "encoder":
        return [(1, 16 * c["l"], n, k, 0.02, "normal") for k, n in ENCODER]
    if fam == "attention":
        l = c["l"]
        return [(HEADS, l, l, HEAD_DIM, 1.0, "normal"), (HEADS, l, HEAD_DIM, l, 1.0, "softmax")]
    return [(1, c["m"], c["n"], c["k"], 0.02, "normal")]


def _inputs(case, seed):
    """The operand pairs (A, B) of a pass, made on the GPU from the seed alone."""
    dt = DTYPES[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def uniform(shape):
        return torch.rand(shape, generator=gen, device="cuda").mul_(2.0).sub_(1.0).to(dt)

    def normal(shape, std):
        return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(dt)

    if case["family"] == "conv":
        x = normal((case["n"], case["hw"], case["hw"], case["cin"]), 1.0)
        return [(x, normal((case["f"], case["f"], case["cin"], case["cout"]), 0.05))]
    pairs = []
    for batch, m, n, k, std, kind in _products(case):
        head = (batch,) if batch > 1 else ()
        if kind == "uniform":
            pairs.append((uniform(head + (m, k)), uniform(head + (k, n))))
        elif kind == "softmax":
            p = torch.softmax(torch.randn(head + (m, k), generator=gen, device="cuda"), dim=-1).to(dt)
            pairs.append((p, normal(head + (k, n), std)))
        else:
            pairs.append((normal(head + (m, k), 1.0), normal(head + (k, n), std)))
    return pairs


def prepare(case, seed):
    state = {"case": case, "pairs": _inputs(case, seed)}
    if case.get("entry") == "abi":
        a, b = state["pairs"][0]
        state["out"] = torch.empty((a.shape[0], b.shape[1]), dtype=a.dtype, device=a.device)
    return state


def run(state):
    case = state["case"]
    if case["family"] == "conv":
        x, w = state["pairs"][0]
        s, p = case["stride"], case["pad"]
        return vx.conv2d(x, w, stride=(s, s), padding=(p, p))
    if case.get("entry") == "abi":
        a, b = state["pairs"][0]
        out = state["out"]
        st = vx.vx_gemm(a.shape[0], b.shape[1], a.shape[1], ABI_CODES[case["dtype"]], a.data_ptr(), b.data_ptr(),
                        out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        if st != 0:
            raise RuntimeError(vx.vx_status_string(st))
        return out
    if case["family"] == "attention":
        return [vx.bmm(a, b) for a, b in state["pairs"]]
    outs = [vx.gemm(a, b) for a, b in state["pairs"]]
    return outs if len(outs) > 1 else outs[0]


def work(case):
    eb = 4 if case["dtype"] == "f32" else 2
    if case["family"] == "conv":
        o, f = _out_dim(case), case["f"]
        pixels = case["n"] * o * o
        taps = f * f * case["cin"]
        return {"bytes": eb * (case["n"] * case["hw"] ** 2 * case["cin"] + taps * case["cout"] + pixels * case["cout"]),
                "flops": 2 * pixels * taps * case["cout"]}
    ps = _products(case)
    return {"bytes": sum(eb * b * (m * k + k * n + m * n) for b, m, n, k, _, _ in ps),
            "flops": sum(2 * b * m * n * k for b, m, n, k, _, _ in ps)}


def tolerance(case):
    # Products are accumulated in fp32 and rounded once into the output type.
    # Measured against `exact` over the listed cases: fp16 2.1e-4 and bf16
    # 1.7e-3 (the rounding of the result), fp32 5e-7 at K = 768 (its sums; they
    # grow as the root of K, which goes to 4096); the largest single difference
    # is one unit in the last place, 2^-10 of the value in fp16 and 2^-7 in bf16.
    return {"f32": {"rel": 4e-6, "max": 4e-5}, "f16": {"rel": 8e-4, "max": 4e-3},
            "bf16": {"rel": 7e-3, "max": 3e-2}}[case["dtype"]]


def exact(case, seed):
    pairs = _inputs(case, seed)
    if case["family"] == "conv":
        x, w = pairs[0]
        f, s, p = case["f"], case["stride"], case["pad"]
        o = _out_dim(case)
        wd = w.double()
        ys = []
        for img in x:    # one tap at a time, an image at a time
            xp = torch.nn.functional.pad(img.double(), (0, 0, p, p, p, p))
            y = torch.zeros((o * o, case["cout"]), dtype=torch.float64, device=x.device)
            for i in range(f):
                for j in range(f):
                    tap = xp[i:i + s * (o - 1) + 1:s, j:j + s * (o - 1) + 1:s]
                    y.addmm_(tap.reshape(o * o, case["cin"]), wd[i, j])
            ys.append(y.view(o, o, case["cout"]))
        return torch.stack(ys)
    if case["family"] == "attention":
        outs = []
        for a, b in pairs:
            outs.append(torch.stack([a[h].double() @ b[h].double() for h in range(a.shape[0])]))
        return outs
    outs = [a.double() @ b.double() for a, b in pairs]
    return outs if len(outs) > 1 else outs[0]
