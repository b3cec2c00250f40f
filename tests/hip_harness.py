"""Helpers that drive libhapi on the GPU through its C ABI for the tests.

Torch only allocates device memory and provides the stream; every step of the
forward pass runs in the library.  Inputs come from ``synth``; expected values
come from the oracle, computed on the CPU from the same synthetic arrays.
"""
from __future__ import annotations

import json
import os
import tempfile

import numpy as np
import torch

import paper_2210_08650_amd as H
import synth


def rel_l2(y, ref) -> float:
    y = np.asarray(y, np.float64)
    ref = np.asarray(ref, np.float64)
    den = np.linalg.norm(ref.ravel())
    return float(np.linalg.norm((y - ref).ravel()) / (den if den > 0 else 1.0))


def bf16_round(x) -> np.ndarray:
    """Round to bfloat16 (nearest even) and widen back to float32."""
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).float().numpy()


def images_for(dtype: int, imgs_f32: np.ndarray):
    """(device tensor in the model dtype, float32 values the oracle should see)."""
    if dtype == H.HAPI_BF16:
        t = torch.from_numpy(np.ascontiguousarray(imgs_f32, np.float32)).to(torch.bfloat16)
        return t.cuda(), t.float().numpy()
    t = torch.from_numpy(np.ascontiguousarray(imgs_f32, np.float32))
    return t.cuda(), imgs_f32.astype(np.float32)


GUARD = 4096        # bytes of sentinel before and after every output and workspace
SENTINEL = 0xA5     # byte pattern of the sentinel


class Guarded:
    """A device buffer with GUARD bytes of sentinel on both sides, plus the
    library's own guard gaps inside a workspace; check() fails if a kernel
    wrote into any of them."""

    def __init__(self, nbytes, inner_gaps=()):
        self.nbytes = int(nbytes)
        self.raw = torch.full((self.nbytes + 2 * GUARD + 256,), SENTINEL, dtype=torch.uint8, device="cuda")
        off = (-self.raw.data_ptr()) % 256 + GUARD     # 256-byte aligned body
        self.off = off
        self.body = self.raw[off:off + self.nbytes]
        self.gaps = [(0, off), (off + self.nbytes, self.raw.numel())] + \
                    [(off + g, off + g + H.HAPI_GUARD_BYTES) for g in inner_gaps]

    def view(self, dtype, shape):
        return self.body.view(dtype).view(shape)

    def check(self):
        for a, b in self.gaps:
            seg = self.raw[a:b]
            bad = int((seg != SENTINEL).sum())
            assert bad == 0, f"{bad} bytes written into the guard [{a - self.off}, {b - self.off}) " \
                             f"of a {self.nbytes}-byte buffer"


def kernel_names(call):
    """Names of the library's kernels that ``call`` launches, e.g.
    ``conv_bf16_ws2_kernel<64, 64, 2, 2, 4, 1, 1, 2, false>``, in launch order."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        call()
        torch.cuda.synchronize()
    names = []
    for e in sorted(p.events(), key=lambda e: e.time_range.start):
        if "hapi::" in e.name:
            n = e.name.removeprefix("void ").replace("hapi::", "").replace("(anonymous namespace)::", "")
            names.append(n.replace("(Loader)", "").split("(")[0])
    return names


def kernel_grids(call):
    """(name up to its template arguments, workgroups) of the library's kernels that ``call`` launches."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        call()
        torch.cuda.synchronize()
    with tempfile.TemporaryDirectory() as d:
        p.export_chrome_trace(os.path.join(d, "trace.json"))
        with open(os.path.join(d, "trace.json")) as f:
            events = json.load(f)["traceEvents"]
    return [(e["name"].removeprefix("void ").replace("hapi::", "").replace("(anonymous namespace)::", "")
             .split("<")[0].split("(")[0], int(np.prod(e["args"]["grid"])))
            for e in events if e.get("cat") == "kernel" and "hapi::" in e["name"]]


def assert_routes(call, wanted=(), unwanted=()):
    """``call`` launches a kernel whose name starts with each of ``wanted`` and none
    that starts with one of ``unwanted``.  The tile rules count tiles against CUs,
    so this holds for the 256-CU device the cases are made for.  The tracer can drop
    records: three tries for it to see them all."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        return
    for _ in range(3):
        names = kernel_names(call)
        bad = [n for n in names if any(n.startswith(u) for u in unwanted)]
        missing = [w for w in wanted if not any(n.startswith(w) for n in names)]
        assert not bad, (bad, names)
        if names and not missing:
            return
    raise AssertionError(f"kernels {missing} not among {names}")


class Runner:
    """A packed model resident on the GPU, ready for repeated extraction."""

    def __init__(self, layers, dtype, params, in_shape=(3, 224, 224)):
        self.layers, self.dtype, self.in_shape = layers, dtype, tuple(in_shape)
        self.stream = torch.cuda.current_stream()
        # direct launches: each call here uses fresh buffers, so none would
        # replay a captured graph anyway (plan replay has a test of its own)
        self.desc = H.Desc(layers, dtype, in_shape, stream=self.stream, direct=1)
        raw = torch.from_numpy(synth.flatten(params)).cuda()
        assert raw.numel() == H.hapi_raw_weight_count(self.desc)
        # zeroed, so that the alignment gaps the packer skips compare equal
        self.packed = torch.zeros(max(H.hapi_packed_weight_bytes(self.desc), 256),
                                  dtype=torch.uint8, device="cuda")
        H.hapi_pack_weights(self.desc, raw if raw.numel() else None, self.packed)
        torch.cuda.synchronize()
        del raw
        self.tdtype = torch.bfloat16 if dtype == H.HAPI_BF16 else torch.float32

    def out_shape(self, split):
        return H.hapi_layer_shape(self.desc, split)

    def _buffers(self, batch, split, chunk, inflight, workspace_pad=0):
        """Guarded workspace and output: every call checks that no kernel
        wrote outside its output, its workspace regions or its workspace."""
        self.desc.set(chunk=chunk, inflight=inflight)
        need = H.hapi_workspace_bytes(self.desc, batch, split)
        ws = Guarded(max(need + workspace_pad, 256), H.hapi_workspace_guards(self.desc, batch, split))
        self.desc.set(workspace=ws.body, workspace_bytes=need + workspace_pad)
        shape = (batch,) + self.out_shape(split)
        out = Guarded(int(np.prod(shape)) * (2 if self.tdtype == torch.bfloat16 else 4))
        return ws, out, out.view(self.tdtype, shape)

    def extract(self, images_dev, split, chunk=0, workspace_pad=0, out=None, inflight=0):
        batch = images_dev.shape[0]
        ws, gout, o = self._buffers(batch, split, chunk, inflight, workspace_pad)
        H.hapi_extract(self.desc, self.packed, images_dev, batch, split, o if out is None else out)
        torch.cuda.synchronize()
        ws.check()
        if out is not None:
            return out
        gout.check()
        return o.clone()

    def resume(self, input_dev, start, end, chunk=0, inflight=0):
        """Layers start+1..end on the layer-``start`` tensor (caller layout)."""
        batch = input_dev.shape[0]
        ws, gout, o = self._buffers(batch, end, chunk, inflight)
        H.hapi_extract_range(self.desc, self.packed, input_dev, batch, start, end, o)
        torch.cuda.synchronize()
        ws.check()
        gout.check()
        return o.clone()

    def extract_np(self, images_dev, split, chunk=0, inflight=0):
        return self.extract(images_dev, split, chunk, inflight=inflight).float().cpu().numpy()
