"""ctypes binding of libcryosplat (argument marshalling only).

Every computation runs in the HIP library; this module checks tensor
placement, dtype and contiguity, packs the C structs declared in
``include/cryosplat.h`` and passes device pointers plus the current torch
stream.  It raises if the shared library is missing: there is no fallback.
"""
from __future__ import annotations

import ctypes
import dataclasses
import os
import threading
from typing import Optional

import numpy as np
import torch

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libcryosplat.so")

CS_SUM, CS_MEAN = 0, 1
_SCALE_ACT = {"exp": 0, "softplus": 1}
_AMP_ACT = {"identity": 0, "softplus": 1}


class CsGaussians(ctypes.Structure):
    _fields_ = [("means", ctypes.c_void_p), ("log_scales", ctypes.c_void_p),
                ("quats", ctypes.c_void_p), ("amps", ctypes.c_void_p),
                ("n", ctypes.c_int64), ("scale_act", ctypes.c_int32),
                ("amp_act", ctypes.c_int32)]


class CsViews(ctypes.Structure):
    _fields_ = [("rot", ctypes.c_void_p), ("shift", ctypes.c_void_p), ("b", ctypes.c_int64),
                ("d", ctypes.c_int32), ("pixel", ctypes.c_float)]


class CsCtf(ctypes.Structure):
    _fields_ = [("defocus_u", ctypes.c_void_p), ("defocus_v", ctypes.c_void_p),
                ("astig", ctypes.c_void_p), ("phase", ctypes.c_void_p),
                ("voltage_kv", ctypes.c_double), ("cs_mm", ctypes.c_double),
                ("amp_contrast", ctypes.c_double), ("bfactor", ctypes.c_double),
                ("pixel_a", ctypes.c_float)]


class CsDataset(ctypes.Structure):
    _fields_ = [("images", ctypes.c_void_p), ("rot", ctypes.c_void_p), ("m", ctypes.c_int64),
                ("d", ctypes.c_int32), ("pixel", ctypes.c_float)]


class CsGrads(ctypes.Structure):
    _fields_ = [("means", ctypes.c_void_p), ("log_scales", ctypes.c_void_p),
                ("quats", ctypes.c_void_p), ("amps", ctypes.c_void_p),
                ("rot", ctypes.c_void_p), ("shift", ctypes.c_void_p)]


_GRAD_SHAPES = {"means": lambda n, b: (n, 3), "log_scales": lambda n, b: (n, 3),
                "quats": lambda n, b: (n, 4), "amps": lambda n, b: (n,),
                "rot": lambda n, b: (b, 3, 3), "shift": lambda n, b: (b, 2)}


def _grads_struct(grads, dev, n, b):
    """CsGrads of a dict of output tensors (missing or None keys are skipped)."""
    return CsGrads(*(_ptr(grads.get(k), k, dev, _GRAD_SHAPES[k](n, b)) for k in
                     ("means", "log_scales", "quats", "amps", "rot", "shift")))


class CsOptions(ctypes.Structure):
    _fields_ = [("q_cut", ctypes.c_float), ("tile", ctypes.c_int32), ("halo", ctypes.c_int32),
                ("budget", ctypes.c_int32), ("graph", ctypes.c_int32),
                ("lane_order", ctypes.c_int32)]


class CsProblem(ctypes.Structure):
    _fields_ = [("g", CsGaussians), ("v", CsViews), ("ctf", ctypes.POINTER(CsCtf)),
                ("opt", CsOptions), ("observed", ctypes.c_void_p), ("reduction", ctypes.c_int32),
                ("loss", ctypes.c_void_p), ("grads", CsGrads), ("images_out", ctypes.c_void_p)]


#: Entry points declared in include/cryosplat.h.
EXPORTS = ("cs_create", "cs_destroy", "cs_last_error", "cs_render", "cs_render_backward",
           "cs_loss_and_grad", "cs_loss_and_grad_noalloc", "cs_loss_and_grad_multi",
           "cs_autotune", "cs_adam_step",
           "cs_pair_count", "cs_set_timing", "cs_stage_time", "cs_set_debug_checks",
           "cs_cnn_create", "cs_cnn_destroy", "cs_cnn_param_count", "cs_cnn_get_params",
           "cs_cnn_set_params", "cs_cnn_forward", "cs_cnn_forward_std", "cs_cnn_train_step",
           "cs_bf16_conv3x3s2_forward", "cs_bf16_conv3x3s2_dgrad", "cs_bf16_conv3x3s2_wgrad",
           "cs_bf16_linear_forward", "cs_bf16_linear_dgrad", "cs_bf16_linear_wgrad",
           "cs_pose_head", "cs_pose_grid", "cs_pose_bank_create", "cs_pose_bank_destroy",
           "cs_pose_bank_size", "cs_pose_bank_rotations", "cs_pose_grid_search", "cs_pose_refine", "cs_add_noise", "cs_cnn_tensor",
           "cs_pose_batch_create", "cs_pose_batch_destroy", "cs_pose_batch_load",
           "cs_pose_batch_search", "cs_pose_batch_refine", "cs_pose_batch_confidence",
           "cs_ctf_filter",
           "cs_voxelize", "cs_fsc", "cs_fsc_resolution", "cs_fourier_shift",
           "cs_init_attributes", "cs_train_sequential", "cs_split_gaussians")


class CryoSplatError(RuntimeError):
    pass


class NonFiniteError(CryoSplatError):
    """A call under debug checks found NaN or infinity (status CS_ERR_NONFINITE)."""


#: status codes of include/cryosplat.h
CS_ERR_INVALID_ARG, CS_ERR_UNSUPPORTED, CS_ERR_OOM, CS_ERR_HIP, CS_ERR_NONFINITE = -1, -2, -3, -4, -5


def load_library(path: str = LIB_PATH) -> ctypes.CDLL:
    """dlopen libcryosplat.so and declare its signatures (no GPU needed)."""
    if not os.path.exists(path):
        raise CryoSplatError(
            f"{path} is missing: build it with paper_2508_04929_amd.build.build() "
            "(the renderer has no CPU fallback)")
    lib = ctypes.CDLL(path)
    vp, i32, i64, f32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float
    P = ctypes.POINTER
    lib.cs_create.argtypes = [ctypes.c_int, P(vp)]
    lib.cs_create.restype = ctypes.c_int
    lib.cs_destroy.argtypes = [vp]
    lib.cs_destroy.restype = None
    lib.cs_last_error.argtypes = [vp]
    lib.cs_last_error.restype = ctypes.c_char_p
    lib.cs_render.argtypes = [vp, P(CsGaussians), P(CsViews), P(CsCtf), P(CsOptions), vp, vp]
    lib.cs_render.restype = ctypes.c_int
    lib.cs_render_backward.argtypes = [vp, P(CsGaussians), P(CsViews), P(CsCtf), P(CsOptions), vp,
                                       P(CsGrads), vp]
    lib.cs_render_backward.restype = ctypes.c_int
    lib.cs_loss_and_grad.argtypes = [vp, P(CsGaussians), P(CsViews), P(CsCtf), P(CsOptions), vp,
                                     i32, vp, P(CsGrads), vp, vp]
    lib.cs_loss_and_grad.restype = ctypes.c_int
    lib.cs_loss_and_grad_noalloc.argtypes = lib.cs_loss_and_grad.argtypes
    lib.cs_loss_and_grad_noalloc.restype = ctypes.c_int
    lib.cs_loss_and_grad_multi.argtypes = [vp, P(CsProblem), i32, i32, vp]
    lib.cs_loss_and_grad_multi.restype = ctypes.c_int
    lib.cs_autotune.argtypes = [vp, P(CsProblem), i32, i32, vp]
    lib.cs_autotune.restype = ctypes.c_int
    lib.cs_adam_step.argtypes = [vp, vp, vp, vp, vp, i64, i64, f32, f32, f32, f32, vp]
    lib.cs_adam_step.restype = ctypes.c_int
    lib.cs_pair_count.argtypes = [vp, P(CsGaussians), P(CsViews), P(CsOptions), vp, vp]
    lib.cs_pair_count.restype = ctypes.c_int
    lib.cs_set_timing.argtypes = [vp, ctypes.c_int]
    lib.cs_set_timing.restype = ctypes.c_int
    lib.cs_stage_time.argtypes = [vp, ctypes.c_char_p, P(ctypes.c_double), P(i64)]
    lib.cs_stage_time.restype = ctypes.c_int
    u64 = ctypes.c_uint64
    lib.cs_cnn_create.argtypes = [vp, i32, i32, u64, P(vp)]
    lib.cs_cnn_destroy.argtypes = [vp]
    lib.cs_cnn_destroy.restype = None
    lib.cs_cnn_param_count.argtypes = [vp]
    lib.cs_cnn_param_count.restype = i64
    lib.cs_cnn_get_params.argtypes = [vp, vp, vp]
    lib.cs_cnn_set_params.argtypes = [vp, vp, vp]
    lib.cs_cnn_forward.argtypes = [vp, vp, i32, vp, vp, vp, vp]
    lib.cs_cnn_forward_std.argtypes = [vp, vp, i32, vp, vp, vp, vp]
    lib.cs_cnn_train_step.argtypes = [vp, vp, vp, vp, i32, f32, f32, vp, vp, i32, vp]
    lib.cs_bf16_conv3x3s2_forward.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32, i32, i32, vp, vp,
                                              vp]
    lib.cs_bf16_conv3x3s2_dgrad.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32, i32, vp, vp, vp]
    lib.cs_bf16_conv3x3s2_wgrad.argtypes = [vp, vp, vp, i32, i32, i32, i32, i32, vp, vp]
    lib.cs_bf16_linear_forward.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32, vp, vp, vp]
    lib.cs_bf16_linear_dgrad.argtypes = [vp, vp, vp, vp, i32, i32, i32, vp, vp, vp]
    lib.cs_bf16_linear_wgrad.argtypes = [vp, vp, vp, i32, i32, i32, vp, vp]
    lib.cs_pose_head.argtypes = [vp, vp, i32, vp, vp, vp, vp, f32, vp, vp, vp]
    lib.cs_pose_grid.argtypes = [i32, i32, vp, P(i64)]
    lib.cs_pose_bank_create.argtypes = [vp, P(CsGaussians), vp, i64, i32, i32, f32, P(CsOptions),
                                        P(vp), vp]
    lib.cs_pose_bank_destroy.argtypes = [vp]
    lib.cs_pose_bank_destroy.restype = None
    lib.cs_pose_bank_size.argtypes = [vp]
    lib.cs_pose_bank_size.restype = i64
    lib.cs_pose_bank_rotations.argtypes = [vp, vp, vp]
    lib.cs_pose_grid_search.argtypes = [vp, vp, P(CsCtf), i32, i32, vp, vp, vp, vp, vp]
    lib.cs_pose_refine.argtypes = [vp, vp, P(CsCtf), i32, vp, i32, i32, i32, vp, vp, vp, vp, vp, vp]
    lib.cs_add_noise.argtypes = [vp, vp, i32, i32, f32, u64, i64, vp]
    lib.cs_cnn_tensor.argtypes = [vp, i32, i32, vp, i64, vp]
    lib.cs_pose_batch_create.argtypes = [vp, i32, f32, i32, i32, P(vp)]
    lib.cs_pose_batch_destroy.argtypes = [vp]
    lib.cs_pose_batch_destroy.restype = None
    lib.cs_pose_batch_load.argtypes = [vp, vp, P(CsCtf), i32, vp, vp, vp]
    lib.cs_pose_batch_search.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp]
    lib.cs_voxelize.argtypes = [vp, P(CsGaussians), i32, f32, f32, vp, vp]
    lib.cs_set_debug_checks.argtypes = [vp, ctypes.c_int]
    lib.cs_set_debug_checks.restype = ctypes.c_int
    lib.cs_fsc.argtypes = [vp, vp, vp, i32, vp, vp]
    lib.cs_fsc_resolution.argtypes = [vp, vp, i32, f32, f32, vp, vp, vp]
    lib.cs_fourier_shift.argtypes = [vp, vp, vp, i64, i32, f32, f32, vp, vp]
    lib.cs_init_attributes.argtypes = [vp, vp, i64, vp, vp]
    lib.cs_split_gaussians.argtypes = [vp, vp, vp, vp, i64, i32, i32, vp, vp, vp, vp]
    lib.cs_train_sequential.argtypes = [vp, vp, vp, vp, i64, i32, i32, P(CsDataset), P(CsCtf),
                                        P(CsOptions), i32, vp, i64, i64, f32, f32, f32, f32, vp,
                                        vp]
    lib.cs_pose_batch_refine.argtypes = [vp, vp, vp, i32, i32, vp, vp, vp, vp, vp, vp, vp]
    lib.cs_pose_batch_confidence.argtypes = [vp, vp, vp, vp, vp, vp, vp]
    lib.cs_ctf_filter.argtypes = [vp, vp, P(CsCtf), i32, i32, f32, vp, vp]
    for name in ("cs_pose_batch_create", "cs_pose_batch_load", "cs_pose_batch_search",
                 "cs_pose_batch_refine", "cs_pose_batch_confidence", "cs_ctf_filter",
                 "cs_voxelize", "cs_fsc",
                 "cs_fsc_resolution", "cs_fourier_shift", "cs_init_attributes", "cs_train_sequential",
                 "cs_split_gaussians", "cs_cnn_tensor", "cs_add_noise", "cs_pose_grid", "cs_pose_bank_create", "cs_pose_bank_rotations",
                 "cs_pose_grid_search", "cs_pose_refine"):
        getattr(lib, name).restype = ctypes.c_int
    for name in ("cs_cnn_create", "cs_cnn_get_params", "cs_cnn_set_params", "cs_cnn_forward",
                 "cs_cnn_train_step", "cs_bf16_conv3x3s2_forward", "cs_bf16_conv3x3s2_dgrad",
                 "cs_bf16_conv3x3s2_wgrad", "cs_bf16_linear_forward", "cs_bf16_linear_dgrad",
                 "cs_bf16_linear_wgrad", "cs_pose_head"):
        getattr(lib, name).restype = ctypes.c_int
    return lib


@dataclasses.dataclass
class Ctf:
    """Per-image CTF parameters as device tensors [B] plus microscope scalars."""
    defocus_u: torch.Tensor
    defocus_v: torch.Tensor
    astig: Optional[torch.Tensor] = None
    phase: Optional[torch.Tensor] = None
    voltage_kv: float = 300.0
    cs_mm: float = 2.7
    amp_contrast: float = 0.1
    bfactor: float = 0.0
    pixel_a: float = 0.0  # Angstrom pixel of the CTF grid when the geometry uses other units


@dataclasses.dataclass
class Options:
    q_cut: float = 0.0   # <= 0: library default 2 ln 1e6
    tile: int = 0
    halo: int = 0
    budget: int = 0
    graph: int = 0       # 1: capture/replay the call as a HIP graph
    lane_order: int = 0  # 1: dealt by LDS bank, 2: sorted by footprint shape (same results)


@dataclasses.dataclass
class Problem:
    """One independent problem of a batched call (device tensors).

    ``loss`` [B+1] and the gradient tensors are outputs; they are allocated
    by :meth:`Library.make_problem` and reused across calls so that a
    captured graph stays valid.
    """
    means: torch.Tensor
    log_scales: torch.Tensor
    quats: torch.Tensor
    amps: torch.Tensor
    rot: torch.Tensor
    shift: Optional[torch.Tensor]
    D: int
    pixel: float
    observed: torch.Tensor
    ctf: Optional[Ctf] = None
    options: Optional[Options] = None
    reduction: str = "sum"
    loss: Optional[torch.Tensor] = None
    grads: Optional[dict] = None
    images_out: Optional[torch.Tensor] = None
    scale_act: str = "exp"
    amp_act: str = "identity"


def _ptr(t: Optional[torch.Tensor], name: str, device, shape=None, dtype=torch.float32):
    if t is None:
        return None
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a torch.Tensor")
    if t.device != device:
        raise ValueError(f"{name} is on {t.device}, expected {device}")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
    return t.data_ptr()


class Library:
    """One libcryosplat context per device, created lazily."""

    def __init__(self, lib: ctypes.CDLL):
        self.lib = lib
        self._ctx = {}
        self._lock = threading.Lock()

    def ctx(self, device: torch.device):
        idx = device.index if device.index is not None else torch.cuda.current_device()
        with self._lock:
            if idx not in self._ctx:
                h = ctypes.c_void_p()
                rc = self.lib.cs_create(idx, ctypes.byref(h))
                if rc != 0:
                    raise CryoSplatError(f"cs_create({idx}) failed with status {rc}")
                self._ctx[idx] = h
            return self._ctx[idx]

    def _check(self, ctx, rc, what):
        if rc != 0:
            msg = self.lib.cs_last_error(ctx).decode(errors="replace")
            cls = NonFiniteError if rc == CS_ERR_NONFINITE else CryoSplatError
            raise cls(f"{what} failed ({rc}): {msg}")

    # -- struct packing -------------------------------------------------
    @staticmethod
    def _pack(means, log_scales, quats, amps, rot, shift, D, pixel, ctf, options,
              scale_act, amp_act):
        dev = rot.device
        n = means.shape[0]
        b = rot.shape[0]
        g = CsGaussians(_ptr(means, "means", dev, (n, 3)), _ptr(log_scales, "log_scales", dev, (n, 3)),
                        _ptr(quats, "quats", dev, (n, 4)), _ptr(amps, "amps", dev, (n,)), n,
                        _SCALE_ACT[scale_act], _AMP_ACT[amp_act])
        v = CsViews(_ptr(rot, "rot", dev, (b, 3, 3)), _ptr(shift, "shift", dev, (b, 2)), b, int(D),
                    float(pixel))
        c = None
        if ctf is not None:
            c = _ctf_struct(ctf, b, dev)
        o = None
        if options is not None:
            o = CsOptions(float(options.q_cut), int(options.tile), int(options.halo),
                          int(options.budget), int(options.graph), int(options.lane_order))
        return dev, n, b, g, v, c, o

    @staticmethod
    def _ref(s):
        return ctypes.byref(s) if s is not None else None

    # -- entry points ----------------------------------------------------
    def render(self, means, log_scales, quats, amps, rot, shift, D, pixel, ctf=None,
               options=None, scale_act="exp", amp_act="identity", out=None):
        dev, n, b, g, v, c, o = self._pack(means, log_scales, quats, amps, rot, shift, D, pixel,
                                           ctf, options, scale_act, amp_act)
        if out is None:
            out = torch.empty((b, D, D), device=dev, dtype=torch.float32)
        _ptr(out, "images", dev, (b, D, D))
        ctx = self.ctx(dev)
        rc = self.lib.cs_render(ctx, ctypes.byref(g), ctypes.byref(v), self._ref(c), self._ref(o),
                                out.data_ptr(), torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_render")
        return out

    def voxelize(self, means, log_scales, quats, amps, D, pixel, q_cut=0.0, scale_act="exp",
                 amp_act="identity", out=None):
        """The mixture's density on a D^3 grid [iz][iy][ix] (cs_voxelize)."""
        dev = means.device
        n = means.shape[0]
        g = CsGaussians(_ptr(means, "means", dev, (n, 3)), _ptr(log_scales, "log_scales", dev, (n, 3)),
                        _ptr(quats, "quats", dev, (n, 4)), _ptr(amps, "amps", dev, (n,)), n,
                        _SCALE_ACT[scale_act], _AMP_ACT[amp_act])
        if out is None:
            out = torch.empty((D, D, D), device=dev, dtype=torch.float32)
        _ptr(out, "vol", dev, (D, D, D))
        ctx = self.ctx(dev)
        self._check(ctx, self.lib.cs_voxelize(ctx, ctypes.byref(g), int(D), float(pixel),
                                              float(q_cut), out.data_ptr(),
                                              torch.cuda.current_stream(dev).cuda_stream),
                    "cs_voxelize")
        return out

    def fsc(self, vol_a, vol_b, out=None):
        """Fourier shell correlation per shell 0 .. D/2 (cs_fsc)."""
        dev = vol_a.device
        D = vol_a.shape[0]
        _ptr(vol_a, "vol_a", dev, (D, D, D))
        _ptr(vol_b, "vol_b", dev, (D, D, D))
        if out is None:
            out = torch.empty(D // 2 + 1, device=dev, dtype=torch.float32)
        _ptr(out, "fsc", dev, (D // 2 + 1,))
        ctx = self.ctx(dev)
        self._check(ctx, self.lib.cs_fsc(ctx, vol_a.data_ptr(), vol_b.data_ptr(), int(D),
                                         out.data_ptr(), torch.cuda.current_stream(dev).cuda_stream),
                    "cs_fsc")
        return out

    def fourier_shift(self, images, shift, pixel, direction=1, out=None):
        """Translate images [B][D][D] by direction * shift [B][2] (band-limited,
        circular; cs_fourier_shift).  direction = -1 centres them."""
        dev = images.device
        B, D = images.shape[0], images.shape[-1]
        _ptr(images, "images", dev, (B, D, D))
        _ptr(shift, "shift", dev, (B, 2))
        if out is None:
            out = torch.empty_like(images)
        _ptr(out, "out", dev, (B, D, D))
        ctx = self.ctx(dev)
        self._check(ctx, self.lib.cs_fourier_shift(ctx, images.data_ptr(), shift.data_ptr(), B, int(D),
                                                   float(pixel), float(direction), out.data_ptr(),
                                                   torch.cuda.current_stream(dev).cuda_stream),
                    "cs_fourier_shift")
        return out

    def init_attributes(self, z, out=None):
        """Flat initial pre-activation parameters [11 N] from normal draws
        z [N][3] (cs_init_attributes)."""
        dev = z.device
        n = z.shape[0]
        _ptr(z, "z", dev, (n, 3))
        if out is None:
            out = torch.empty(11 * n, device=dev, dtype=torch.float32)
        _ptr(out, "params", dev, (11 * n,))
        ctx = self.ctx(dev)
        self._check(ctx, self.lib.cs_init_attributes(ctx, z.data_ptr(), n, out.data_ptr(),
                                                     torch.cuda.current_stream(dev).cuda_stream),
                    "cs_init_attributes")
        return out

    def split_gaussians(self, params, adam_m=None, adam_v=None, scale_act="softplus",
                        amp_act="softplus", out=None):
        """Densify: flat parameters [11 N] -> [22 N] (and the Adam moments when
        given), cs_split_gaussians.  Returns (params, m, v); `out` may hold
        the three [22 N] output tensors (None entries are allocated)."""
        dev = params.device
        np_ = params.numel()
        if np_ % 11:
            raise ValueError("params must hold 11 values per Gaussian")
        n = np_ // 11
        _ptr(params, "params", dev, (np_,))
        mom = adam_m is not None or adam_v is not None
        o_p, o_m, o_v = out if out is not None else (None, None, None)
        out = o_p if o_p is not None else torch.empty(2 * np_, device=dev, dtype=torch.float32)
        _ptr(out, "out", dev, (2 * np_,))
        om = ov = None
        if mom:
            _ptr(adam_m, "adam_m", dev, (np_,))
            _ptr(adam_v, "adam_v", dev, (np_,))
            om = o_m if o_m is not None else torch.empty_like(out)
            ov = o_v if o_v is not None else torch.empty_like(out)
            _ptr(om, "out_m", dev, (2 * np_,))
            _ptr(ov, "out_v", dev, (2 * np_,))
        ctx = self.ctx(dev)
        rc = self.lib.cs_split_gaussians(
            ctx, params.data_ptr(), adam_m.data_ptr() if mom else None,
            adam_v.data_ptr() if mom else None, n, _SCALE_ACT[scale_act], _AMP_ACT[amp_act],
            out.data_ptr(), om.data_ptr() if mom else None, ov.data_ptr() if mom else None,
            torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_split_gaussians")
        return out, om, ov

    def train_sequential(self, params, adam_m, adam_v, images, rot, pixel, order, step0, lr,
                         ctf=None, options=None, reduction="sum", b1=0.9, b2=0.999, eps=1e-8,
                         scale_act="softplus", amp_act="softplus", loss=None):
        """Batch-1 steps of Alg. 1 over the images in ``order`` (host int64
        indices) on flat parameters [11 N] (cs_train_sequential)."""
        dev = params.device
        np_ = params.numel()
        if np_ % 11:
            raise ValueError("params must hold 11 values per Gaussian")
        n = np_ // 11
        for t, nm in ((params, "params"), (adam_m, "adam_m"), (adam_v, "adam_v")):
            _ptr(t, nm, dev, (np_,))
        M, D = images.shape[0], images.shape[-1]
        data = CsDataset(_ptr(images, "images", dev, (M, D, D)), _ptr(rot, "rot", dev, (M, 3, 3)),
                         M, int(D), float(pixel))
        order = np.ascontiguousarray(order, dtype=np.int64)
        c = _ctf_struct(ctf, M, dev)
        o = None
        if options is not None:
            o = CsOptions(float(options.q_cut), int(options.tile), int(options.halo),
                          int(options.budget), int(options.graph), int(options.lane_order))
        if loss is not None:
            _ptr(loss, "loss", dev, (len(order),))
        ctx = self.ctx(dev)
        red = {"sum": 0, "mean": 1}[reduction]
        rc = self.lib.cs_train_sequential(
            ctx, params.data_ptr(), adam_m.data_ptr(), adam_v.data_ptr(), n, _SCALE_ACT[scale_act],
            _AMP_ACT[amp_act], ctypes.byref(data), self._ref(c), self._ref(o), red,
            order.ctypes.data_as(ctypes.c_void_p), len(order), int(step0), float(lr), float(b1),
            float(b2), float(eps), loss.data_ptr() if loss is not None else None,
            torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_train_sequential")
        return loss

    def resolution(self, fsc, D, pixel, threshold=0.143):
        """Resolution read-out of an FSC curve on the device (cs_fsc_resolution):
        returns (resolution in Angstrom, shell index) as host numbers."""
        dev = fsc.device
        _ptr(fsc, "fsc", dev, (D // 2 + 1,))
        out = torch.empty(2, device=dev, dtype=torch.float32)
        ctx = self.ctx(dev)
        shell = out[1:].view(torch.int32)
        self._check(ctx, self.lib.cs_fsc_resolution(
            ctx, fsc.data_ptr(), int(D), float(pixel), float(threshold), shell.data_ptr(),
            out.data_ptr(), torch.cuda.current_stream(dev).cuda_stream), "cs_fsc_resolution")
        h = out.cpu()
        return float(h[0]), int(h[1:].view(torch.int32)[0])

    def _grads(self, dev, n, b, pose=False):
        """Fresh gradient outputs: the Gaussian parameters, and with pose the
        views' rotations [B][3][3] and shifts [B][2]."""
        z = lambda *s: torch.empty(s, device=dev, dtype=torch.float32)
        gr = {"means": z(n, 3), "log_scales": z(n, 3), "quats": z(n, 4), "amps": z(n)}
        if pose:
            gr.update(rot=z(b, 3, 3), shift=z(b, 2))
        return gr, _grads_struct(gr, dev, n, b)

    def render_backward(self, means, log_scales, quats, amps, rot, shift, D, pixel, d_images,
                        ctf=None, options=None, scale_act="exp", amp_act="identity",
                        want_pose_grads=False):
        dev, n, b, g, v, c, o = self._pack(means, log_scales, quats, amps, rot, shift, D, pixel,
                                           ctf, options, scale_act, amp_act)
        _ptr(d_images, "d_images", dev, (b, D, D))
        gr, cg = self._grads(dev, n, b, want_pose_grads)
        ctx = self.ctx(dev)
        rc = self.lib.cs_render_backward(ctx, ctypes.byref(g), ctypes.byref(v), self._ref(c),
                                         self._ref(o), d_images.data_ptr(), ctypes.byref(cg),
                                         torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_render_backward")
        return gr

    def loss_and_grad(self, means, log_scales, quats, amps, rot, shift, D, pixel, observed,
                      ctf=None, options=None, reduction="sum", want_grads=True,
                      want_images=False, scale_act="exp", amp_act="identity", grads=None,
                      loss=None, want_pose_grads=False, images=None, noalloc=False):
        """Loss per image (+ total) and gradients; with want_pose_grads the
        gradients also hold "rot" [B][3][3] and "shift" [B][2]; a caller's
        grads dict may hold any subset of the six outputs.  With
        noalloc=True the call goes to cs_loss_and_grad_noalloc (the library's
        static scratch; pass preallocated loss, grads and images to keep the
        whole call free of allocations)."""
        dev, n, b, g, v, c, o = self._pack(means, log_scales, quats, amps, rot, shift, D, pixel,
                                           ctf, options, scale_act, amp_act)
        _ptr(observed, "observed", dev, (b, D, D))
        if loss is None:
            loss = torch.empty(b + 1, device=dev, dtype=torch.float32)
        _ptr(loss, "loss", dev, (b + 1,))
        cg = None
        if want_grads:
            if grads is None:
                grads, cg = self._grads(dev, n, b, want_pose_grads)
            else:
                cg = _grads_struct(grads, dev, n, b)
        if images is not None:
            _ptr(images, "images", dev, (b, D, D))
        elif want_images:
            images = torch.empty((b, D, D), device=dev, dtype=torch.float32)
        ctx = self.ctx(dev)
        fn = self.lib.cs_loss_and_grad_noalloc if noalloc else self.lib.cs_loss_and_grad
        rc = fn(ctx, ctypes.byref(g), ctypes.byref(v), self._ref(c), self._ref(o),
                observed.data_ptr(), CS_MEAN if reduction == "mean" else CS_SUM, loss.data_ptr(),
                self._ref(cg), images.data_ptr() if images is not None else None,
                torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_loss_and_grad_noalloc" if noalloc else "cs_loss_and_grad")
        return loss, (grads if want_grads else None), images

    # -- batched problems -------------------------------------------------
    def make_problem(self, means, log_scales, quats, amps, rot, shift, D, pixel, observed,
                     ctf=None, options=None, reduction="sum", want_grads=True, want_images=False,
                     scale_act="exp", amp_act="identity", want_pose_grads=False) -> Problem:
        dev = rot.device
        n, b = means.shape[0], rot.shape[0]
        z = lambda *s: torch.zeros(s, device=dev, dtype=torch.float32)
        grads = ({"means": z(n, 3), "log_scales": z(n, 3), "quats": z(n, 4), "amps": z(n)}
                 if want_grads else None)
        if grads is not None and want_pose_grads:
            grads.update(rot=z(b, 3, 3), shift=z(b, 2))
        return Problem(means, log_scales, quats, amps, rot, shift, D, pixel, observed, ctf,
                       options or Options(), reduction, z(b + 1), grads,
                       z(b, D, D) if want_images else None, scale_act, amp_act)

    def _problem_struct(self, pr: Problem):
        dev, n, b, g, v, c, o = self._pack(pr.means, pr.log_scales, pr.quats, pr.amps, pr.rot,
                                           pr.shift, pr.D, pr.pixel, pr.ctf,
                                           pr.options or Options(), pr.scale_act, pr.amp_act)
        _ptr(pr.observed, "observed", dev, (b, pr.D, pr.D))
        _ptr(pr.loss, "loss", dev, (b + 1,))
        cg = CsGrads()
        if pr.grads is not None:
            cg = _grads_struct(pr.grads, dev, n, b)
        io = _ptr(pr.images_out, "images_out", dev, (b, pr.D, pr.D)) if pr.images_out is not None else None
        s = CsProblem(g, v, ctypes.pointer(c) if c is not None else None, o, pr.observed.data_ptr(),
                      CS_MEAN if pr.reduction == "mean" else CS_SUM, pr.loss.data_ptr(), cg, io)
        return dev, s, c

    def _problem_array(self, problems):
        structs, keep, dev = [], [], None
        for pr in problems:
            dev, s, c = self._problem_struct(pr)
            structs.append(s)
            keep.append(c)
        arr = (CsProblem * len(structs))(*structs)
        return dev, arr, keep

    def loss_and_grad_multi(self, problems, use_graph=True):
        """All problems' losses and gradients in one batched call (writes pr.loss / pr.grads)."""
        dev, arr, keep = self._problem_array(problems)
        ctx = self.ctx(dev)
        rc = self.lib.cs_loss_and_grad_multi(ctx, arr, len(problems), 1 if use_graph else 0,
                                             torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_loss_and_grad_multi")
        del keep
        return problems

    def autotune(self, problems, reps=2):
        """Choose tile/halo/budget per problem (writes pr.options)."""
        dev, arr, keep = self._problem_array(problems)
        ctx = self.ctx(dev)
        rc = self.lib.cs_autotune(ctx, arr, len(problems), int(reps),
                                  torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_autotune")
        for pr, s in zip(problems, arr):
            base = pr.options or Options()
            pr.options = Options(q_cut=base.q_cut, tile=s.opt.tile, halo=s.opt.halo,
                                 budget=s.opt.budget, graph=base.graph,
                                 lane_order=s.opt.lane_order)
        del keep
        return problems

    def adam_step(self, params, grads, m, v, step, lr=1e-3, b1=0.9, b2=0.999, eps=1e-8):
        dev = params.device
        for t, nm in ((params, "params"), (grads, "grads"), (m, "m"), (v, "v")):
            _ptr(t, nm, dev, tuple(params.shape))
        ctx = self.ctx(dev)
        rc = self.lib.cs_adam_step(ctx, params.data_ptr(), grads.data_ptr(), m.data_ptr(),
                                   v.data_ptr(), params.numel(), int(step), float(lr), float(b1),
                                   float(b2), float(eps), torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_adam_step")

    def pair_count(self, means, log_scales, quats, amps, rot, shift, D, pixel, options=None,
                   scale_act="exp"):
        dev, n, b, g, v, c, o = self._pack(means, log_scales, quats, amps, rot, shift, D, pixel,
                                           None, options, scale_act, "identity")
        out = torch.empty(b, device=dev, dtype=torch.int64)
        ctx = self.ctx(dev)
        rc = self.lib.cs_pair_count(ctx, ctypes.byref(g), ctypes.byref(v), self._ref(o),
                                    out.data_ptr(), torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_pair_count")
        return out


    def set_debug_checks(self, device, enable: bool):
        """Debug checks: calls scan their inputs and outputs for NaN / infinity,
        synchronise, and fail with status CS_ERR_NONFINITE (NonFiniteError)."""
        dev = self._device(device)
        self._check(self.ctx(dev), self.lib.cs_set_debug_checks(self.ctx(dev), int(bool(enable))),
                    "cs_set_debug_checks")

    def set_timing(self, device, enable: bool):
        ctx = self.ctx(torch.device(device))
        self._check(ctx, self.lib.cs_set_timing(ctx, 1 if enable else 0), "cs_set_timing")

    def stage_time(self, device, name: str):
        """(total milliseconds, launches) of one library stage since timing was enabled."""
        ctx = self.ctx(torch.device(device))
        ms, n = ctypes.c_double(), ctypes.c_int64()
        self._check(ctx, self.lib.cs_stage_time(ctx, name.encode(), ctypes.byref(ms), ctypes.byref(n)),
                    "cs_stage_time")
        return ms.value, n.value

    def add_noise(self, images, snr_db, seed, offset=0):
        """In place: images [B][D][D] += white noise at snr_db per image."""
        dev = images.device
        B, D = images.shape[0], images.shape[1]
        _ptr(images, "images", dev, (B, D, D))
        ctx = self.ctx(dev)
        rc = self.lib.cs_add_noise(ctx, images.data_ptr(), B, D, float(snr_db), int(seed),
                                   int(offset), torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_add_noise")
        return images

    # -- pose scoring ------------------------------------------------------
    def pose_grid(self, nside: int, n_psi: int):
        """HEALPix x psi rotation grid (host float32 [K][3][3])."""
        import numpy as np
        n = ctypes.c_int64()
        rc = self.lib.cs_pose_grid(int(nside), int(n_psi), None, ctypes.byref(n))
        if rc != 0:
            raise CryoSplatError(f"cs_pose_grid({nside}, {n_psi}) failed ({rc})")
        out = np.empty((n.value, 3, 3), dtype=np.float32)
        rc = self.lib.cs_pose_grid(int(nside), int(n_psi), out.ctypes.data, ctypes.byref(n))
        if rc != 0:
            raise CryoSplatError(f"cs_pose_grid failed ({rc})")
        return out

    def pose_bank(self, means, log_scales, quats, amps, rot, n_psi, D, pixel, options=None,
                  scale_act="exp", amp_act="identity"):
        K = rot.shape[0]
        dev, n, b, g, v, c, o = self._pack(means, log_scales, quats, amps, rot, None, D, pixel,
                                           None, options, scale_act, amp_act)
        ctx = self.ctx(dev)
        h = ctypes.c_void_p()
        rc = self.lib.cs_pose_bank_create(ctx, ctypes.byref(g), rot.data_ptr(), K, int(n_psi),
                                          int(D), float(pixel), self._ref(o), ctypes.byref(h),
                                          torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_pose_bank_create")
        return PoseBank(self, self._device(dev), h, K, D, pixel, n_psi)

    def pose_batch(self, D: int, pixel: float, capacity: int, shift_radius: int = 2,
                   device="cuda"):
        return PoseBatch(self, self._device(device), D, pixel, capacity, shift_radius)

    def ctf_filter(self, images, ctf, pixel, out=None):
        """out = F^-1(H^ F images) per image (ApplyCTF); out may be images."""
        dev = images.device
        B, D = images.shape[0], images.shape[1]
        _ptr(images, "images", dev, (B, D, D))
        if out is None:
            out = torch.empty_like(images)
        _ptr(out, "out", dev, (B, D, D))
        c = _ctf_struct(ctf, B, dev)
        ctx = self.ctx(dev)
        rc = self.lib.cs_ctf_filter(ctx, images.data_ptr(), None if c is None else ctypes.byref(c),
                                    B, D, float(pixel), out.data_ptr(),
                                    torch.cuda.current_stream(dev).cuda_stream)
        self._check(ctx, rc, "cs_ctf_filter")
        return out

    # -- pose-proposal network -------------------------------------------
    @staticmethod
    def _device(device) -> torch.device:
        d = torch.device(device)
        return torch.device(d.type, d.index if d.index is not None else torch.cuda.current_device())

    def network(self, D: int, max_batch: int, seed: int = 0, device="cuda"):
        return Network(self, self._device(device), D, max_batch, seed)

    def _stream(self, dev):
        return torch.cuda.current_stream(dev).cuda_stream

    def conv_forward(self, x, w, bias, relu=True, want_f32=False):
        """x [B][H][W][Cin] bf16, w [Cout][3][3][Cin] bf16 -> (y bf16, y_f32 or None)."""
        dev = x.device
        B, H, W, Cin = x.shape
        Cout = w.shape[0]
        _ptr(x, "x", dev, dtype=torch.bfloat16)
        _ptr(w, "w", dev, (Cout, 3, 3, Cin), dtype=torch.bfloat16)
        _ptr(bias, "bias", dev, (Cout,))
        y = torch.empty(B, H // 2, W // 2, Cout, device=dev, dtype=torch.bfloat16)
        y32 = torch.empty(y.shape, device=dev) if want_f32 else None
        ctx = self.ctx(dev)
        rc = self.lib.cs_bf16_conv3x3s2_forward(ctx, x.data_ptr(), w.data_ptr(),
                                                 None if bias is None else bias.data_ptr(), B, H, W,
                                                 Cin, Cout, int(relu), y.data_ptr(),
                                                 None if y32 is None else y32.data_ptr(),
                                                 self._stream(dev))
        self._check(ctx, rc, "cs_bf16_conv3x3s2_forward")
        return y, y32

    def conv_dgrad(self, dy, wt, act_in, want_f32=False):
        """dy [B][H/2][W/2][Cout], wt [Cin][3][3][Cout] -> dx [B][H][W][Cin] (bf16)."""
        dev = dy.device
        B, Ho, Wo, Cout = dy.shape
        Cin = wt.shape[0]
        H, W = 2 * Ho, 2 * Wo
        _ptr(dy, "dy", dev, dtype=torch.bfloat16)
        _ptr(wt, "wt", dev, (Cin, 3, 3, Cout), dtype=torch.bfloat16)
        _ptr(act_in, "act_in", dev, (B, H, W, Cin), dtype=torch.bfloat16)
        dx = torch.empty(B, H, W, Cin, device=dev, dtype=torch.bfloat16)
        dx32 = torch.empty(dx.shape, device=dev) if want_f32 else None
        ctx = self.ctx(dev)
        rc = self.lib.cs_bf16_conv3x3s2_dgrad(ctx, dy.data_ptr(), wt.data_ptr(),
                                               None if act_in is None else act_in.data_ptr(), B, H,
                                               W, Cin, Cout, dx.data_ptr(),
                                               None if dx32 is None else dx32.data_ptr(),
                                               self._stream(dev))
        self._check(ctx, rc, "cs_bf16_conv3x3s2_dgrad")
        return dx, dx32

    def conv_wgrad(self, dy, x):
        """dy [B][H/2][W/2][Cout], x [B][H][W][Cin] -> dw [Cout][3][3][Cin] FP32."""
        dev = dy.device
        B, H, W, Cin = x.shape
        Cout = dy.shape[-1]
        _ptr(dy, "dy", dev, (B, H // 2, W // 2, Cout), dtype=torch.bfloat16)
        _ptr(x, "x", dev, dtype=torch.bfloat16)
        dw = torch.empty(Cout, 3, 3, Cin, device=dev)
        ctx = self.ctx(dev)
        rc = self.lib.cs_bf16_conv3x3s2_wgrad(ctx, dy.data_ptr(), x.data_ptr(), B, H, W, Cin, Cout,
                                               dw.data_ptr(), self._stream(dev))
        self._check(ctx, rc, "cs_bf16_conv3x3s2_wgrad")
        return dw

    def linear_forward(self, x, w, bias, relu=True, want_bf16=True):
        """x [B][In] bf16, w [Out][In] bf16 -> (y bf16 or None, y FP32)."""
        dev = x.device
        B, In = x.shape
        Out = w.shape[0]
        _ptr(x, "x", dev, dtype=torch.bfloat16)
        _ptr(w, "w", dev, (Out, In), dtype=torch.bfloat16)
        _ptr(bias, "bias", dev, (Out,))
        y = torch.empty(B, Out, device=dev, dtype=torch.bfloat16) if want_bf16 else None
        y32 = torch.empty(B, Out, device=dev)
        ctx = self.ctx(dev)
        rc = self.lib.cs_bf16_linear_forward(ctx, x.data_ptr(), w.data_ptr(),
                                              None if bias is None else bias.data_ptr(), B, In, Out,
                                              int(relu), None if y is None else y.data_ptr(),
                                              y32.data_ptr(), self._stream(dev))
        self._check(ctx, rc, "cs_bf16_linear_forward")
        return y, y32

    def linear_dgrad(self, dy, wt, x_act, want_f32=False):
        dev = dy.device
        B, Out = dy.shape
        In = wt.shape[0]
        _ptr(dy, "dy", dev, dtype=torch.bfloat16)
        _ptr(wt, "wt", dev, (In, Out), dtype=torch.bfloat16)
        _ptr(x_act, "x_act", dev, (B, In), dtype=torch.bfloat16)
        dx = torch.empty(B, In, device=dev, dtype=torch.bfloat16)
        dx32 = torch.empty(B, In, device=dev) if want_f32 else None
        ctx = self.ctx(dev)
        rc = self.lib.cs_bf16_linear_dgrad(ctx, dy.data_ptr(), wt.data_ptr(),
                                            None if x_act is None else x_act.data_ptr(), B, In, Out,
                                            dx.data_ptr(), None if dx32 is None else dx32.data_ptr(),
                                            self._stream(dev))
        self._check(ctx, rc, "cs_bf16_linear_dgrad")
        return dx, dx32

    def linear_wgrad(self, dy, x):
        dev = dy.device
        B, Out = dy.shape
        In = x.shape[1]
        _ptr(dy, "dy", dev, dtype=torch.bfloat16)
        _ptr(x, "x", dev, (B, In), dtype=torch.bfloat16)
        dw = torch.empty(Out, In, device=dev)
        ctx = self.ctx(dev)
        rc = self.lib.cs_bf16_linear_wgrad(ctx, dy.data_ptr(), x.data_ptr(), B, In, Out,
                                            dw.data_ptr(), self._stream(dev))
        self._check(ctx, rc, "cs_bf16_linear_wgrad")
        return dw

    def pose_head(self, raw, rot_target=None, shift_target=None, lam=1.0):
        """raw [B][8] -> dict(rot [B][3][3], shift [B][2], and with targets loss, d_raw)."""
        dev = raw.device
        B = raw.shape[0]
        _ptr(raw, "raw", dev, (B, 8))
        rot = torch.empty(B, 3, 3, device=dev)
        shift = torch.empty(B, 2, device=dev)
        out = {"rot": rot, "shift": shift}
        args = [None, None, None, None]
        if rot_target is not None:
            _ptr(rot_target, "rot_target", dev, (B, 3, 3))
            _ptr(shift_target, "shift_target", dev, (B, 2))
            out["loss"] = torch.empty(1, device=dev)
            out["d_raw"] = torch.empty(B, 8, device=dev)
            args = [rot_target.data_ptr(), shift_target.data_ptr(), out["loss"].data_ptr(),
                    out["d_raw"].data_ptr()]
        ctx = self.ctx(dev)
        rc = self.lib.cs_pose_head(ctx, raw.data_ptr(), B, rot.data_ptr(), shift.data_ptr(),
                                   args[0], args[1], float(lam), args[2], args[3],
                                   self._stream(dev))
        self._check(ctx, rc, "cs_pose_head")
        return out


class PoseBank:
    """Handle of a cs_pose_bank (projections + power spectra of a rotation set)."""

    def __init__(self, owner: "Library", device: torch.device, h, K: int, D: int, pixel: float,
                 n_psi: int):
        self.owner, self.lib, self.device = owner, owner.lib, device
        self.ctx = owner.ctx(device)
        self.h, self.K, self.D, self.pixel, self.n_psi = h, K, D, pixel, n_psi

    def close(self):
        if getattr(self, "h", None) is not None and self.h.value:
            self.lib.cs_pose_bank_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _s(self):
        return torch.cuda.current_stream(self.device).cuda_stream

    def rotations(self):
        out = torch.empty(self.K, 3, 3, device=self.device)
        self.owner._check(self.ctx, self.lib.cs_pose_bank_rotations(self.h, out.data_ptr(), self._s()),
                          "cs_pose_bank_rotations")
        return out

    def _ctf(self, ctf, P):
        if ctf is None:
            return None
        return _ctf_struct(ctf, P, self.device)

    def _outs(self, P, S, ncols, want_scores):
        d = self.device
        out = {"rot_idx": torch.empty(P, device=d, dtype=torch.int32),
               "shift_idx": torch.empty(P, device=d, dtype=torch.int32),
               "score": torch.empty(P, device=d)}
        out["scores"] = torch.empty(P, ncols, S, device=d) if want_scores else None
        return out

    @staticmethod
    def _p(t):
        return None if t is None else t.data_ptr()

    def grid_search(self, images, ctf=None, shift_radius=2, want_scores=False):
        P = images.shape[0]
        _ptr(images, "images", self.device, (P, self.D, self.D))
        S = (2 * shift_radius + 1) ** 2
        out = self._outs(P, S, self.K, want_scores)
        c = self._ctf(ctf, P)
        self.owner._check(self.ctx, self.lib.cs_pose_grid_search(
            self.h, images.data_ptr(), None if c is None else ctypes.byref(c), P, int(shift_radius),
            out["rot_idx"].data_ptr(), out["shift_idx"].data_ptr(), out["score"].data_ptr(),
            self._p(out["scores"]), self._s()), "cs_pose_grid_search")
        return out

    def refine(self, images, ctf=None, proposal=None, cand=None, n_dir=8, n_psi_c=3,
               shift_radius=2, want_scores=False):
        P = images.shape[0]
        _ptr(images, "images", self.device, (P, self.D, self.D))
        S = (2 * shift_radius + 1) ** 2
        if proposal is None:
            if cand is None:
                raise ValueError("need a proposal or candidate lists")
            L = cand.shape[1]
            n_dir, n_psi_c = L, 1
        else:
            _ptr(proposal, "proposal", self.device, (P, 3, 3))
            L = n_dir * n_psi_c
            if cand is None:
                cand = torch.empty(P, L, device=self.device, dtype=torch.int32)
        _ptr(cand, "cand", self.device, (P, L), dtype=torch.int32)
        out = self._outs(P, S, L, want_scores)
        out["cand"] = cand
        c = self._ctf(ctf, P)
        self.owner._check(self.ctx, self.lib.cs_pose_refine(
            self.h, images.data_ptr(), None if c is None else ctypes.byref(c), P,
            self._p(proposal), int(n_dir), int(n_psi_c), int(shift_radius), cand.data_ptr(),
            out["rot_idx"].data_ptr(), out["shift_idx"].data_ptr(), out["score"].data_ptr(),
            self._p(out["scores"]), self._s()), "cs_pose_refine")
        return out


def _ctf_struct(ctf, P, device):
    if ctf is None:
        return None
    return CsCtf(_ptr(ctf.defocus_u, "defocus_u", device, (P,)),
                 _ptr(ctf.defocus_v, "defocus_v", device, (P,)),
                 _ptr(ctf.astig, "astig", device, (P,)), _ptr(ctf.phase, "phase", device, (P,)),
                 float(ctf.voltage_kv), float(ctf.cs_mm), float(ctf.amp_contrast),
                 float(ctf.bfactor), float(ctf.pixel_a))


class PoseBatch:
    """Handle of a cs_pose_batch: particle-side data shared by searches."""

    def __init__(self, owner: "Library", device: torch.device, D: int, pixel: float,
                 capacity: int, shift_radius: int):
        self.owner, self.lib, self.device = owner, owner.lib, device
        self.ctx = owner.ctx(device)
        self.D, self.pixel, self.capacity, self.r = D, pixel, capacity, shift_radius
        self.S = (2 * shift_radius + 1) ** 2
        h = ctypes.c_void_p()
        owner._check(self.ctx, self.lib.cs_pose_batch_create(self.ctx, D, float(pixel), capacity,
                                                             shift_radius, ctypes.byref(h)),
                     "cs_pose_batch_create")
        self.h, self.P = h, 0

    def close(self):
        if getattr(self, "h", None) is not None and self.h.value:
            self.lib.cs_pose_batch_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _s(self):
        return torch.cuda.current_stream(self.device).cuda_stream

    def load(self, images, ctf=None, filtered=None, standardized=None):
        """Prepare P images; filtered [P][D][D] FP32 (optional) receives Z = H Y,
        standardized [P][D][D] bfloat16 (optional) the network input (Z
        standardised per image)."""
        P = images.shape[0]
        _ptr(images, "images", self.device, (P, self.D, self.D))
        _ptr(filtered, "filtered", self.device, (P, self.D, self.D))
        _ptr(standardized, "standardized", self.device, (P, self.D, self.D), torch.bfloat16)
        c = _ctf_struct(ctf, P, self.device)
        self.owner._check(self.ctx, self.lib.cs_pose_batch_load(
            self.h, images.data_ptr(), None if c is None else ctypes.byref(c), P,
            None if filtered is None else filtered.data_ptr(),
            None if standardized is None else standardized.data_ptr(), self._s()),
            "cs_pose_batch_load")
        self.P = P
        return filtered

    def _outs(self, ncols, want_scores):
        d, P = self.device, self.P
        return {"rot_idx": torch.empty(P, device=d, dtype=torch.int32),
                "shift_idx": torch.empty(P, device=d, dtype=torch.int32),
                "score": torch.empty(P, device=d),
                "rot": torch.empty(P, 3, 3, device=d),
                "scores": torch.empty(P, ncols, self.S, device=d) if want_scores else None}

    def search(self, bank: "PoseBank", want_scores=False):
        out = self._outs(bank.K, want_scores)
        self.owner._check(self.ctx, self.lib.cs_pose_batch_search(
            bank.h, self.h, out["rot_idx"].data_ptr(), out["shift_idx"].data_ptr(),
            out["score"].data_ptr(), PoseBank._p(out["scores"]), out["rot"].data_ptr(), self._s()),
            "cs_pose_batch_search")
        return out

    def refine(self, bank: "PoseBank", proposal=None, cand=None, n_dir=8, n_psi_c=3,
               want_scores=False):
        P = self.P
        if proposal is None:
            if cand is None:
                raise ValueError("need a proposal or candidate lists")
            L = cand.shape[1]
            n_dir, n_psi_c = L, 1
        else:
            _ptr(proposal, "proposal", self.device, (P, 3, 3))
            L = n_dir * n_psi_c
        if cand is not None:
            _ptr(cand, "cand", self.device, (P, L), dtype=torch.int32)
        out = self._outs(L, want_scores)
        out["cand"] = cand
        self.owner._check(self.ctx, self.lib.cs_pose_batch_refine(
            bank.h, self.h, PoseBank._p(proposal), int(n_dir), int(n_psi_c), PoseBank._p(cand),
            out["rot_idx"].data_ptr(), out["shift_idx"].data_ptr(), out["score"].data_ptr(),
            PoseBank._p(out["scores"]), out["rot"].data_ptr(), self._s()), "cs_pose_batch_refine")
        return out


    def confidence(self, bank: "PoseBank", out, z=None, sigmas=None, want_sigmas=False):
        """Fit statistic z [P] of the winning poses in `out` (a search or
        refinement result of this batch on `bank`): 2 a - 1 with a the
        least-squares amplitude of the winning template in the particle.
        With want_sigmas (or a sigmas tensor) also the shortfall (1 - z) in
        units of z's noise spread; returns (z, sigmas) then."""
        P = self.P
        _ptr(out["rot_idx"], "rot_idx", self.device, (P,), torch.int32)
        _ptr(out["score"], "score", self.device, (P,))
        if z is None:
            z = torch.empty(P, device=self.device)
        _ptr(z, "z", self.device, (P,))
        if sigmas is None and want_sigmas:
            sigmas = torch.empty(P, device=self.device)
        _ptr(sigmas, "sigmas", self.device, (P,))
        self.owner._check(self.ctx, self.lib.cs_pose_batch_confidence(
            bank.h, self.h, out["rot_idx"].data_ptr(), out["score"].data_ptr(), z.data_ptr(),
            PoseBank._p(sigmas), self._s()), "cs_pose_batch_confidence")
        return (z, sigmas) if sigmas is not None else z


class Network:
    """Handle of a cs_cnn pose-proposal network (owned; freed on close/del)."""

    def __init__(self, owner: Library, device: torch.device, D: int, max_batch: int, seed: int):
        self.owner, self.lib, self.device = owner, owner.lib, device
        self.D, self.max_batch = D, max_batch
        self.ctx = owner.ctx(device)
        h = ctypes.c_void_p()
        owner._check(self.ctx, self.lib.cs_cnn_create(self.ctx, D, max_batch, int(seed),
                                                      ctypes.byref(h)), "cs_cnn_create")
        self.h = h
        self.n_params = int(self.lib.cs_cnn_param_count(self.h))

    def close(self):
        if getattr(self, "h", None) is not None and self.h.value:
            self.lib.cs_cnn_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _s(self):
        return torch.cuda.current_stream(self.device).cuda_stream

    def get_params(self):
        out = torch.empty(self.n_params, device=self.device)
        self.owner._check(self.ctx, self.lib.cs_cnn_get_params(self.h, out.data_ptr(), self._s()),
                          "cs_cnn_get_params")
        return out

    def set_params(self, p):
        _ptr(p, "params", self.device, (self.n_params,))
        self.owner._check(self.ctx, self.lib.cs_cnn_set_params(self.h, p.data_ptr(), self._s()),
                          "cs_cnn_set_params")

    def forward(self, images):
        B = images.shape[0]
        _ptr(images, "images", self.device, (B, self.D, self.D))
        rot = torch.empty(B, 3, 3, device=self.device)
        shift = torch.empty(B, 2, device=self.device)
        raw = torch.empty(B, 8, device=self.device)
        self.owner._check(self.ctx, self.lib.cs_cnn_forward(self.h, images.data_ptr(), B,
                                                            rot.data_ptr(), shift.data_ptr(),
                                                            raw.data_ptr(), self._s()),
                          "cs_cnn_forward")
        return rot, shift, raw

    def forward_standardized(self, x):
        """Inference from a standardised bfloat16 input [B][D][D] (PoseBatch.load)."""
        B = x.shape[0]
        _ptr(x, "x", self.device, (B, self.D, self.D), torch.bfloat16)
        rot = torch.empty(B, 3, 3, device=self.device)
        shift = torch.empty(B, 2, device=self.device)
        raw = torch.empty(B, 8, device=self.device)
        self.owner._check(self.ctx, self.lib.cs_cnn_forward_std(self.h, x.data_ptr(), B,
                                                                rot.data_ptr(), shift.data_ptr(),
                                                                raw.data_ptr(), self._s()),
                          "cs_cnn_forward_std")
        return rot, shift, raw

    def tensor(self, index: int, grad: bool, shape):
        """Stored bfloat16 activation (grad=False) or gradient (grad=True) of the last call."""
        out = torch.empty(shape, device=self.device, dtype=torch.bfloat16)
        self.owner._check(self.ctx, self.lib.cs_cnn_tensor(self.h, int(index), int(grad),
                                                           out.data_ptr(), out.numel(), self._s()),
                          "cs_cnn_tensor")
        return out

    def train_step(self, images, rot_target, shift_target, lam=1.0, lr=1e-3, update=True,
                   want_grads=False, loss=None):
        B = images.shape[0]
        _ptr(images, "images", self.device, (B, self.D, self.D))
        _ptr(rot_target, "rot_target", self.device, (B, 3, 3))
        _ptr(shift_target, "shift_target", self.device, (B, 2))
        if loss is None:
            loss = torch.empty(1, device=self.device)
        grads = torch.empty(self.n_params, device=self.device) if want_grads else None
        self.owner._check(self.ctx, self.lib.cs_cnn_train_step(
            self.h, images.data_ptr(), rot_target.data_ptr(), shift_target.data_ptr(), B,
            float(lam), float(lr), loss.data_ptr(), None if grads is None else grads.data_ptr(),
            int(update), self._s()), "cs_cnn_train_step")
        return loss, grads


#: Kernel stages the library may launch (names reported by stage_time).
STAGES = ("k_build", "k_bin_count", "k_bin_blockscan", "k_scan", "k_bin_scatter", "k_ctf_table", "k_splat_fwd", "k_canvas_reduce",
          "k_fft_rows_fwd", "k_fft_cols_ctf", "k_fft_rows_inv_loss", "k_fft_rows_inv",
          "k_residual", "k_loss_small", "k_loss_reduce", "k_loss_total", "k_splat_bwd", "k_chain", "k_adam",
          "k_fill", "k_pair_count", "k_pose_grad_part", "k_pose_grad_sum")

_LIB: Optional[Library] = None


#: launch options the autotuner chose on an MI355X for the benchmark
#: workloads (cs_autotune's cache format: signature tile halo budget)
TUNE_DB = os.path.join(HERE, "tune_mi355x.txt")


def use_tune_db(path: str = TUNE_DB) -> None:
    """Point the contexts created from now on at a private copy of a tuning
    database (CS_AUTOTUNE_CACHE): cs_autotune then returns the recorded
    options for known problem signatures without timing, and new entries go
    to the copy, never to the shipped file.  No-op when CS_AUTOTUNE_CACHE is
    already set or the database is missing."""
    if "CS_AUTOTUNE_CACHE" in os.environ or not os.path.exists(path):
        return
    import shutil
    import tempfile
    fd, tmp = tempfile.mkstemp(prefix="cs_tune_", suffix=".txt")
    os.close(fd)
    shutil.copyfile(path, tmp)
    os.environ["CS_AUTOTUNE_CACHE"] = tmp


def library() -> Library:
    """The process-wide binding (loads libcryosplat.so on first use; contexts
    read the shipped tuning database, see use_tune_db)."""
    global _LIB
    if _LIB is None:
        use_tune_db()
        _LIB = Library(load_library())
    return _LIB
