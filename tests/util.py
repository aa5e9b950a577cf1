"""Helpers shared by the GPU parity tests (no method arithmetic here)."""
import os
import subprocess

import numpy as np
import torch

from paper_2509_15148_amd import build as B


def weights_to_numpy(w):
    """Stored weight values as fp32 numpy arrays (bf16 -> fp32 is exact); the oracle widens to fp64."""
    conv = lambda t: t.detach().float().cpu().numpy()
    return {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}


def dev(x, dtype=None):
    t = torch.as_tensor(x)
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda().contiguous()


def ws(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")


def dirty_ws(nbytes):
    """A workspace full of NaN in every type: a value read before it is written shows."""
    return torch.full((max(int(nbytes), 256),), 255, dtype=torch.uint8, device="cuda")


def tight_ws(nbytes):
    """A workspace that ends with its allocation (whole 2 MiB pages of its own): nothing behind it belongs to the process."""
    need = (max(int(nbytes), 256) + 255) // 256 * 256
    page = 2 << 20
    torch.cuda.empty_cache()
    room = torch.empty(-(-max(need, 32 << 20) // page) * page, dtype=torch.uint8, device="cuda")
    return room[room.numel() - need:]


def announce(*what):
    """Name the case before the GPU step runs, flushed, so a lost box still tells which case it was."""
    print("[case]", *what, flush=True)


def device_assembly(src, folder):
    """The assembly of one source file by the build's own flags."""
    path = os.path.join(str(folder), src + ".s")
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", path], check=True, capture_output=True)
    with open(path) as f:
        return f.read()
