"""torch-facing helpers over the C ABI: plan cache, fft / ifft / fft2 /
fft_many, and the differentiable transform.

torch supplies device memory and streams only; every transform runs in the
library's HIP kernels.  Complex64 data are ``torch.complex64`` tensors;
16-bit data are real ``torch.float16`` / ``torch.bfloat16`` tensors with a
trailing dimension of 2 (re, im), since torch has no complex bfloat16.
"""
from __future__ import annotations

import threading
from array import array

import torch

from . import autotune, capi

_DT = {torch.complex64: capi.FFT_C64, torch.float16: capi.FFT_C16F, torch.bfloat16: capi.FFT_C16BF}


class Plan:
    """Owns one library plan handle."""

    def __init__(self, handle: int, kind: str):
        self.handle = handle
        self.kind = kind
        self.workspace = None  # torch tensor backing a caller-owned workspace
        # batched plans whose kernel waits on completion counters (the
        # two-launch kernels never wait)
        self.waits = kind == "many" and capi.fft_plan_info(handle)["pass_variant"][0] not in ("many_flat",
                                                                                               "many_2launch")
        # bytes of scratch that an exec brings: fused 2-D plans run in place
        # without, and with it save the pass that orders the rows; batched
        # plans of the queue kernel by the planner's rule take their queue
        # state with each call, so that calls on several streams may overlap
        self.scratch = 0
        self.scratch_always = False
        if kind == "strided" and capi.fft_plan_info(handle)["pass_variant"][0].startswith("f"):
            self.scratch = capi.fft_workspace_size(handle)

    def __del__(self):
        try:
            capi.fft_destroy(self.handle)
        except Exception:
            pass

    def info(self) -> dict:
        return capi.fft_plan_info(self.handle)

    def exec(self, x: torch.Tensor, out: torch.Tensor, stream: int | None = None) -> None:
        if stream is None:
            try:
                stream = _raw_stream(x.device.index)
            except (TypeError, RuntimeError):
                if x.is_cuda:
                    raise
                raise ValueError("input must be a GPU tensor where no stream is given") from None
            if self.scratch and self.workspace is None and (self.scratch_always or x.data_ptr() == out.data_ptr()):
                ws = _scratch(self.scratch, x.device)
                if ws is not None:
                    capi.fft_exec_ws(self.handle, x.data_ptr(), out.data_ptr(), stream, ws.data_ptr(), self.scratch)
                    return
        capi.fft_exec(self.handle, x.data_ptr(), out.data_ptr(), stream)

    def set_scale(self, s: float) -> None:
        capi.fft_set_scale(self.handle, s)

    def ensure_workspace(self, device) -> None:
        need = capi.fft_workspace_size(self.handle)
        if need and (self.workspace is None or self.workspace.numel() < need):
            self.workspace = torch.empty(need, dtype=torch.uint8, device=device)
            capi.fft_set_workspace(self.handle, self.workspace.data_ptr(), need)


# Scratch of one in-place exec of a fused 2-D plan, which saves the pass that
# orders the rows (4096 x 4096: 94 us against 145; 2 x 2048 x 4096: 88 against
# 137).  Larger batches do without, so that one may fill the memory.
_SCRATCH_MAX = 1 << 30


def _scratch(nbytes: int, device):
    """Memory for one exec on the device's current stream, whose order the
    allocator follows when it hands the memory out again; or None where there
    is none to spare, and under capture, where the memory would have to
    outlive the graph."""
    if nbytes > _SCRATCH_MAX:
        return None
    with torch.cuda.device(device):
        if torch.cuda.is_current_stream_capturing():
            return None
        try:
            return torch.empty(nbytes, dtype=torch.uint8, device=device)
        except torch.cuda.OutOfMemoryError:
            return None


_cache: dict = {}
_lock = threading.Lock()

# the current stream's handle of a device by index: without building a
# torch.cuda.Stream where this torch has the function for it (0.1 us against 1.9)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None) or (
    lambda index: torch.cuda.current_stream(int(index)).cuda_stream)

# Plans by call signature: a repeated call finds its plan with one lookup,
# where checking the shape, looking the tuned schedule up and building the
# plan key took as long as the kernel launch (api.fft of one 1024-point signal
# 8.6 -> 5.0 us of host time; fft_many of 512 lengths 89 -> 14 us, most of it
# the digest of the lengths).  The signature holds the tuner's generation, so
# schedules tuned in this process take effect at once.  The entries are plans
# of _cache and leave with it.
_by_call: dict = {}
_by_call_generation = 0


def _remember(key, value) -> None:
    global _by_call_generation
    with _lock:
        if _by_call_generation != autotune.generation:
            _by_call.clear()
            _by_call_generation = autotune.generation
        _by_call[key] = value


def get_plan(shape, batch: int, dtype: int, direction: int, *, scale=None,
             schedule: str | None = None, device=None) -> Plan:
    """Cached plan for `batch` transforms of `shape` (1 or 2 dims)."""
    dev = torch.cuda.current_device() if device is None else torch.device(device).index
    if schedule is None:
        schedule = autotune.schedule_for(shape, batch, dtype)
    key = ("plan", tuple(int(s) for s in shape), int(batch), dtype, direction, scale, schedule, dev)
    with _lock:
        p = _cache.get(key)
        if p is None:
            with torch.cuda.device(dev):
                h = capi.fft_plan_ex(list(shape), batch, len(shape), dtype, direction, schedule)
                p = Plan(h, "strided")
                if scale is not None:
                    p.set_scale(scale)
            _cache[key] = p
    return p


def get_many_plan(sizes, dtype: int, direction: int, *, scale=None, schedule=None,
                  device=None) -> Plan:
    dev = torch.cuda.current_device() if device is None else torch.device(device).index
    ruled = False
    if schedule is None:
        schedule = autotune.many_schedule_for(sizes, dtype)
        ruled = schedule is None
    key = ("many", tuple(int(s) for s in sizes), dtype, direction, scale, schedule, dev)
    with _lock:
        p = _cache.get(key)
        if p is None:
            with torch.cuda.device(dev):
                h = capi.fft_plan_many_ex([int(s) for s in sizes], dtype, direction, schedule)
                p = Plan(h, "many")
                if ruled and p.info()["pass_variant"][0] == "many_2launch":
                    p.scratch, p.scratch_always = capi.fft_workspace_size(h), True
                if scale is not None:
                    p.set_scale(scale)
            _cache[key] = p
    return p


def clear_cache() -> None:
    with _lock:
        _cache.clear()
        _by_call.clear()


def _check_input(x: torch.Tensor, ndim_fft: int):
    if not x.is_cuda:
        raise ValueError("input must be a GPU tensor (the transforms run in HIP kernels only)")
    if x.dtype == torch.complex64:
        shape = x.shape[x.dim() - ndim_fft:]
        lead = x.shape[:x.dim() - ndim_fft]
    elif x.dtype in (torch.float16, torch.bfloat16):
        if x.shape[-1] != 2:
            raise ValueError("16-bit complex data need a trailing dimension of 2 (re, im)")
        shape = x.shape[x.dim() - 1 - ndim_fft:x.dim() - 1]
        lead = x.shape[:x.dim() - 1 - ndim_fft]
    else:
        raise ValueError(f"unsupported dtype {x.dtype}")
    if len(shape) != ndim_fft:
        raise ValueError("input has too few dimensions")
    batch = 1
    for s in lead:
        batch *= int(s)
    return list(shape), batch


def _call_key(*parts, scale, schedule):
    """Signature of a call, or None where a part is no plain value."""
    if scale is not None and type(scale) not in (float, int) or schedule is not None and type(schedule) is not str:
        return None
    return parts + (scale, type(scale), schedule, autotune.generation)


def _run(x, ndim_fft, inverse, scale, out, schedule):
    inverse = bool(inverse)
    key = _call_key(x.shape, x.dtype, x.device, ndim_fft, inverse, scale=scale, schedule=schedule)
    plan = None if key is None else _by_call.get(key)
    if plan is None:
        shape, batch = _check_input(x, ndim_fft)
        direction = capi.FFT_INVERSE if inverse else capi.FFT_FORWARD
        plan = get_plan(shape, batch, _DT[x.dtype], direction, scale=scale, schedule=schedule, device=x.device)
        if key is not None:
            _remember(key, plan)
    x = x.contiguous()
    if out is None:
        out = torch.empty_like(x)
    elif out.shape != x.shape or out.dtype != x.dtype or not out.is_contiguous():
        raise ValueError("out must be a contiguous tensor of the input's shape and dtype")
    if out.data_ptr() == x.data_ptr() and not plan.scratch:
        plan.ensure_workspace(x.device)
    plan.exec(x, out)
    return out


def fft(x: torch.Tensor, inverse: bool = False, *, scale: float | None = None,
        out: torch.Tensor | None = None, schedule: str | None = None) -> torch.Tensor:
    """1-D transform along the last axis (eq. 1; with inverse=True eq. 2).

    Lengths of 2^15 to 2^24 in place (``out=x``), and longer ones always, go
    through scratch that the plan keeps: such calls of one shape must not
    overlap on several streams."""
    return _run(x, 1, inverse, scale, out, schedule)


def ifft(x: torch.Tensor, **kw) -> torch.Tensor:
    return fft(x, inverse=True, **kw)


def fft2(x: torch.Tensor, inverse: bool = False, *, scale: float | None = None,
         out: torch.Tensor | None = None, schedule: str | None = None) -> torch.Tensor:
    """2-D transform over the last two axes: rows, then columns.  In place
    too, on any streams."""
    return _run(x, 2, inverse, scale, out, schedule)


def ifft2(x: torch.Tensor, **kw) -> torch.Tensor:
    return fft2(x, inverse=True, **kw)


def fft_many(packed: torch.Tensor, sizes, inverse: bool = False, *, scale=None,
             out: torch.Tensor | None = None, schedule: str | None = None) -> torch.Tensor:
    """Independent 1-D transforms of lengths `sizes` packed back to back, in
    one exec (two launches)."""
    inverse = bool(inverse)
    key = None
    if type(sizes) in (list, tuple):
        try:
            lengths = array("q", sizes).tobytes()
            key = _call_key(lengths, packed.shape, packed.dtype, packed.device, inverse, scale=scale,
                            schedule=schedule)
        except (TypeError, OverflowError):
            pass  # lengths that are no integers of 64 bits
    plan = None if key is None else _by_call.get(key)
    if plan is None:
        if not packed.is_cuda:
            raise ValueError("input must be a GPU tensor")
        if packed.dtype not in _DT:
            raise ValueError(f"unsupported dtype {packed.dtype}")
        total = packed.numel() if packed.dtype == torch.complex64 else packed.numel() // 2
        if sum(int(s) for s in sizes) != total:
            raise ValueError("sizes do not add up to the packed length")
        direction = capi.FFT_INVERSE if inverse else capi.FFT_FORWARD
        plan = get_many_plan(sizes, _DT[packed.dtype], direction, scale=scale, schedule=schedule,
                             device=packed.device)
        if key is not None:
            _remember(key, plan)
    packed = packed.contiguous()
    if out is None:
        out = torch.empty_like(packed)
    elif out.shape != packed.shape or out.dtype != packed.dtype or not out.is_contiguous():
        raise ValueError("out must be a contiguous tensor of the packed input's shape and dtype")
    plan.exec(packed, out)
    if plan.waits:
        # kernels whose second passes wait on completion counters: a wait that
        # ran out (e.g. workgroups that were not resident) leaves wrong
        # results, so read the flag (this synchronises)
        if capi.fft_many_watchdog(plan.handle, clear=True) == capi.FFT_ERR_WATCHDOG:
            raise RuntimeError("fft_many: a dependency wait expired; the results are invalid")
    return out


class FFTFunction(torch.autograd.Function):
    """y = F x along the last axis (eq. 1, unscaled), differentiable.

    For a real loss torch passes grad_y = dL/dRe(y) + i dL/dIm(y); since F is
    linear and holomorphic, grad_x = F^H grad_y, the inverse-direction
    transform with scale 1 (the adjoint), run by the same HIP kernels.
    """

    @staticmethod
    def forward(ctx, x):
        if x.dtype != torch.complex64:
            raise ValueError("FFTFunction takes complex64 input")
        return fft(x)

    @staticmethod
    def backward(ctx, g):
        return fft(g.contiguous(), inverse=True, scale=1.0)


def fft_autograd(x: torch.Tensor) -> torch.Tensor:
    return FFTFunction.apply(x)


def variants() -> list:
    out = []
    for i in range(capi.fft_variant_count()):
        d = capi.fft_variant_describe(i)
        d["name"] = capi.fft_variant_name(i)
        out.append(d)
    return out
