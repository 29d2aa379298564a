"""The binding where no GPU is needed: what goes wrong on its way to the library ends in an exception, never in
the end of the process.  Device tensors without storage (FakeTensorMode) stand in for a GPU's; calls run in a child."""
import os
import subprocess
import sys
import textwrap

import pytest

pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import warnings
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
import paper_2406_02540_amd as vq
warnings.simplefilter("ignore")


class Stream:
    cuda_stream = 0


def fake(*shape, dtype=torch.float16):
    return torch.empty(shape, dtype=dtype, device="cuda")


M, N, K = 4, 8, 128
f32, i8, u8 = torch.float32, torch.int8, torch.uint8


def outcome(call):
    try:
        call()
        return "returned"
    except torch.AcceleratorError:   # (an allocation on a given stream asks for the current one: there is no device here)
        return "RuntimeError: no device"
    except Exception as e:
        return type(e).__name__ + ": " + str(e).splitlines()[0]
"""


def child(body):
    from paper_2406_02540_amd import binding
    if not (os.path.exists(binding.LIB_PATH) and os.path.exists(binding.EXT_PATH)):
        from paper_2406_02540_amd import build
        build.build(verbose=False)
    out = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body)], cwd=ROOT, timeout=300,
                         capture_output=True, text=True)
    assert out.returncode == 0, (out.returncode, out.stdout, out.stderr[-2000:])
    return dict(line.split("=", 1) for line in out.stdout.splitlines())


def test_tensors_without_an_address_raise():
    # inside a functorch transform a tensor has no address: asking for it throws
    got = child("""
        with FakeTensorMode():
            st = Stream()
            w, w4, ws = fake(N, K, dtype=i8), fake(N, K // 2, dtype=u8), fake(N, dtype=f32)
            q, s, y, r = fake(M, K, dtype=i8), fake(M, dtype=f32), fake(M, N), fake(M, K)
            wk, amax, rot = fake(4096, dtype=u8), fake(K, dtype=f32), fake(N, K, dtype=f32)
            x, wf = (M, K), (N, K)
            entries = {   # name: (shape and type of the tensor that the transform wraps, the call)
                "quantize_per_token": (x, None, lambda a: vq.vq_quantize_per_token(a, None, q, s, stream=st)),
                "gelu_quantize": (x, None, lambda a: vq.vq_gelu_quantize(a, True, None, q, s, stream=st)),
                "layernorm_quantize": (x, None, lambda a: vq.vq_layernorm_quantize(a, xq=q, x_scale=s, stream=st)),
                "residual_quantize": (x, None, lambda a: vq.vq_residual_quantize(a, r, r=r, xq=q, x_scale=s, stream=st)),
                "hadamard_quantize": (x, None, lambda a: vq.vq_hadamard_quantize(a, None, q, s, stream=st)),
                "quantize_static": (x, None, lambda a: vq.vq_quantize_static(a, 0.5, None, q, stream=st)),
                "channel_absmax": (x, None, lambda a: vq.vq_channel_absmax(a, amax, stream=st)),
                "balance_mask": ((K,), f32, lambda a: vq.vq_balance_mask(a, amax, 0.5, stream=st)),
                "rotate_weight": (wf, f32, lambda a: vq.vq_rotate_weight(a, None, rot, stream=st)),
                "quantize_weight": (wf, f32, lambda a: vq.vq_quantize_weight(a, None, 8, stream=st)),
                "gemm_f16": (x, None, lambda a: vq.vq_gemm_f16(a, fake(N, K), None, y, stream=st)),
                "gemm_w8a8": (x, i8, lambda a: vq.vq_gemm_w8a8(a, s, w, ws, None, y, stream=st)),
                "gemm_w4a8": (x, i8, lambda a: vq.vq_gemm_w4a8(a, s, w4, ws, None, y, stream=st)),
                "linear": (x, None, lambda a: vq.vq_linear(a, None, w, 8, ws, None, y, wk, stream=st)),
                "linear_static": (x, None, lambda a: vq.vq_linear_static(a, None, w, 8, ws, None, y, stream=st)),
                "layernorm_linear": (x, None, lambda a: vq.vq_layernorm_linear(a, w, 8, ws, y=y, workspace=wk, stream=st)),
                "gelu_linear": (x, None, lambda a: vq.vq_gelu_linear(a, w, 8, ws, y=y, workspace=wk, stream=st)),
                "residual_linear": (x, None, lambda a: vq.vq_residual_linear(a, r, w, 8, ws, r=r, y=y, workspace=wk, stream=st)),
                "hadamard_linear": (x, None, lambda a: vq.vq_hadamard_linear(a, None, w, 8, ws, y=y, workspace=wk, stream=st)),
            }
            for name, (shape, dtype, call) in entries.items():
                a = fake(3, *shape, dtype=dtype or torch.float16)
                print(name, outcome(lambda: torch.func.vmap(call)(a)), sep="=", flush=True)
                if a.is_floating_point():
                    print(name + "_grad", outcome(lambda: torch.func.grad(call)(a[0])), sep="=", flush=True)
    """)
    assert len(got) == 19 + 17
    assert all(v.startswith("RuntimeError: ") for v in got.values()), got


def test_sample_lengths_that_round_to_zero_or_exceed_an_int():
    # 2**32 + 4 narrowed to an int is the length that the vectors have; -1 fits, and no vector has that many rows
    got = child("""
        with FakeTensorMode():
            st = Stream()
            x, r, v, w, ws = fake(M, K), fake(M, K), fake(1, K, dtype=f32), fake(N, K, dtype=i8), fake(N, dtype=f32)
            q, s, y, wk = fake(M, K, dtype=i8), fake(M, dtype=f32), fake(M, N), fake(4096, dtype=u8)
            for T in (0.5, -1, 2**31, 2**32, 2**32 + 4, 2**70, -2**40):
                for name, call in {
                    "layernorm_quantize": lambda: vq.vq_layernorm_quantize(x, v, None, T, 1e-6, None, q, s, stream=st),
                    "residual_quantize": lambda: vq.vq_residual_quantize(x, r, v, T, r, None, q, s, stream=st),
                    "layernorm_linear": lambda: vq.vq_layernorm_linear(x, w, 8, ws, None, v, T, y=y, workspace=wk, stream=st),
                    "residual_linear": lambda: vq.vq_residual_linear(x, r, w, 8, ws, v, T, r, y=y, workspace=wk, stream=st),
                }.items():
                    print(f"{name} {T}", outcome(call), sep="=", flush=True)
            print("fits", outcome(lambda: vq.vq_layernorm_quantize(x, v, None, 2**31 - 1, 1e-6, None, q, s, stream=st)), sep="=")
    """)
    assert len(got) == 4 * 7 + 1
    assert "VQ_ERR_NULL" in got.pop("fits")   # (a fake tensor's address is null: the length was accepted)
    for k, v in got.items():
        T = k.split()[1]
        want = {"0.5": "ZeroDivisionError: ", "-1": "ValueError: "}.get(T, f"VqError: vq_{k.split()[0]}: VQ_ERR_SHAPE")
        assert v.startswith(want), (k, v)


def test_numbers_as_float_takes_them():
    got = child("""
        with FakeTensorMode():
            st = Stream()
            x, q, s = fake(M, K), fake(M, K, dtype=i8), fake(M, dtype=f32)
            for text in ("0.5", "half"):
                print("eps " + text, outcome(lambda: vq.vq_layernorm_quantize(x, eps=text, xq=q, x_scale=s, stream=st)), sep="=")
                print("scale " + text, outcome(lambda: vq.vq_quantize_static(x, text, None, q, stream=st)), sep="=")
            print("eps None", outcome(lambda: vq.vq_layernorm_quantize(x, eps=None, xq=q, x_scale=s, stream=st)), sep="=")
    """)
    assert all("VQ_ERR_NULL" in got[k] for k in ("eps 0.5", "scale 0.5")), got   # (accepted: null is the fake address)
    assert all(got[k].startswith("ValueError: ") for k in ("eps half", "scale half")), got
    assert got["eps None"].startswith("TypeError: ")
