"""Helpers for the GPU parity tests: numpy <-> device tensors, error norms."""
import numpy as np


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


def empty_like_dev(a):
    import torch
    return torch.empty(a.shape, dtype=torch.complex128, device="cuda")


def rel_err(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def maxabs_ratio(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def note(msg):
    print(msg, flush=True)


def random_links(V, seed):
    """[V][4][3][3] random SU(3) links made on the device."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    a, b = (torch.randn((V, 4, 3), dtype=torch.complex128, device="cuda", generator=g) for _ in range(2))
    a = a / torch.linalg.vector_norm(a, dim=-1, keepdim=True)
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack([a, b, torch.linalg.cross(a, b, dim=-1).conj()], dim=-2).contiguous()
