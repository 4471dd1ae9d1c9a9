"""ctypes binding of libfr (include/fr.h): argument marshalling only.

Device arrays are torch tensors on the handle's GPU (their data_ptr() is passed through);
host arrays are numpy arrays. Every computation runs in libfr's HIP kernels; if the library is
missing this module raises instead of falling back to anything else.
"""
from __future__ import annotations

import ctypes
import os

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
# FR_LIB_PATH selects another build of the same sources (the host-sanitizer build of build.py)
LIB_PATH = os.environ.get("FR_LIB_PATH") or os.path.join(_HERE, "libfr.so")

FR_OK = 0
ERRORS = {-1: "FR_ERR_ARG", -2: "FR_ERR_MESH", -3: "FR_ERR_HIP", -4: "FR_ERR_OOM",
          -5: "FR_ERR_UNSUPPORTED", -6: "FR_ERR_NONFINITE"}
FLUX = {"rusanov": 0, "roe": 1}
PREC = {"fp64": 0, "fp32": 1}
SCHEME = {"rk4": 0, "lsrk45": 1, "ssprk104": 2}


class FRError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"{ERRORS.get(code, code)}: {msg}")
        self.code = code
        self.name = ERRORS.get(code, str(code))


class fr_mesh_desc(ctypes.Structure):
    _fields_ = [
        ("p", ctypes.c_int32), ("q", ctypes.c_int32), ("n_elem", ctypes.c_int64),
        ("elem_vert", ctypes.c_void_p), ("elem_nodes", ctypes.c_void_p),
        ("gamma", ctypes.c_double), ("prandtl", ctypes.c_double), ("mu", ctypes.c_double),
        ("br2_eta", ctypes.c_double), ("flux", ctypes.c_int32), ("prec", ctypes.c_int32),
        ("check_finite", ctypes.c_int32), ("viscous", ctypes.c_int32),
        ("ref_rho", ctypes.c_double), ("ref_p", ctypes.c_double), ("ldg_tau", ctypes.c_double),
        ("bc_tag", ctypes.c_void_p), ("wall_T", ctypes.c_double),
    ]


_lib = None


def load():
    """Load libfr.so (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2308_06605_amd.build`"
                           " (or __graft_entry__.build()); there is no fallback path")
    # torch ships a HIP runtime with the same soname as the system one libfr links against; the
    # first one loaded serves the whole process, so let torch load and initialise its runtime
    # before libfr, as torch's own GPU calls (streams, allocations) need it
    import torch

    torch.cuda.is_available()
    L = ctypes.CDLL(LIB_PATH)
    P, i32, i64, f64 = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_double
    L.fr_last_error.restype = ctypes.c_char_p
    L.fr_mesh_create.argtypes = [ctypes.POINTER(fr_mesh_desc), P, ctypes.POINTER(P)]
    L.fr_mesh_destroy.argtypes = [P]
    L.fr_set_stream.argtypes = [P, P]
    L.fr_sol_coords.argtypes = [P, P]
    L.fr_set_state.argtypes = [P, P, i32]
    L.fr_get_state.argtypes = [P, P, i32]
    L.fr_residual.argtypes = [P, P, i32]
    L.fr_rk_step.argtypes = [P, f64, i32, i32]
    L.fr_mesh_info.argtypes = [P, ctypes.POINTER(i64), ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(i64)]
    L.fr_profile_stages.argtypes = [P, f64, i32, i32, P]
    L.fr_mesh_geometry_host.argtypes = [ctypes.POINTER(fr_mesh_desc), P, P, P, P, P]
    L.fr_basis_host.argtypes = [i32, P, P, P, P, P]
    L.fr_rk_coefficients.argtypes = [i32, P, P, ctypes.POINTER(ctypes.c_int32)]
    L.fr_kinetic_energy.argtypes = [P, P]
    L.fr_set_body_force.argtypes = [P, P]
    L.fr_set_tiles.argtypes = [P, ctypes.c_int32, ctypes.c_int32]
    L.fr_get_tiles.argtypes = [P, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]
    L.fr_tiles_in_force.argtypes = [P, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]
    L.fr_autotune.argtypes = [P, i32, P]
    L.fr_set_fusion.argtypes = [P, ctypes.c_int32]
    L.fr_get_fusion.argtypes = [P, ctypes.POINTER(ctypes.c_int32)]
    L.fr_part_create.argtypes = [ctypes.POINTER(fr_mesh_desc), P, ctypes.c_int32, P, ctypes.POINTER(P)]
    L.fr_part_destroy.argtypes = [P]
    L.fr_part_host.argtypes = [ctypes.POINTER(fr_mesh_desc), P, ctypes.c_int32, ctypes.c_int32,
                               ctypes.POINTER(i64), ctypes.POINTER(i64), P, P]
    L.fr_part_get_mesh.argtypes = [P, ctypes.c_int32, ctypes.POINTER(P)]
    L.fr_part_elements.argtypes = [P, ctypes.c_int32, ctypes.POINTER(i64), P]
    L.fr_part_set_stream.argtypes = [P, P]
    L.fr_halo_size.argtypes = [P, ctypes.c_int32, ctypes.POINTER(i64), ctypes.POINTER(i64)]
    L.fr_halo_pack.argtypes = [P, ctypes.c_int32, P]
    L.fr_halo_unpack.argtypes = [P, ctypes.c_int32, P]
    L.fr_part_residual.argtypes = [P, P, i32]
    L.fr_part_rk_step.argtypes = [P, f64, i32, i32]
    L.fr_batch_create.argtypes = [P, ctypes.c_int32, P, i32, P, ctypes.POINTER(P)]
    L.fr_batch_create_ex.argtypes = [P, ctypes.c_int32, P, i32, P, ctypes.c_int32, ctypes.POINTER(P)]
    L.fr_batch_step.argtypes = [P, i32]
    L.fr_batch_set_stream.argtypes = [P, P]
    L.fr_batch_destroy.argtypes = [P]
    # learned eddy-viscosity closure
    L.fr_sgs_n_features.argtypes = [i32]
    L.fr_sgs_features.argtypes = [P, P]
    L.fr_set_eddy_viscosity.argtypes = [P, P, i32, f64]
    L.fr_set_sgs_model.argtypes = [P, P, f64, f64]
    L.fr_get_eddy_viscosity.argtypes = [P, P]
    L.fr_mlp_n_params.argtypes = [ctypes.c_int32]
    L.fr_mlp_n_params.restype = i64
    L.fr_mlp_create.argtypes = [ctypes.c_int32, P, P, P, P, ctypes.POINTER(P)]
    L.fr_mlp_destroy.argtypes = [P]
    L.fr_mlp_set_stream.argtypes = [P, P]
    L.fr_mlp_set_params.argtypes = [P, P]
    L.fr_mlp_get_params.argtypes = [P, P]
    L.fr_mlp_get_bf16.argtypes = [P, P, P, P]
    L.fr_mlp_forward.argtypes = [P, P, i64, i64, P]
    L.fr_mlp_loss_grad.argtypes = [P, P, i64, i64, P, P, ctypes.POINTER(f64)]
    L.fr_mlp_train_step.argtypes = [P, P, i64, i64, P, ctypes.c_float, P]
    L.fr_mlp_train_step_noalloc.argtypes = [P, P, i64, i64, P, ctypes.c_float, P]
    for name in ("fr_mesh_create", "fr_mesh_destroy", "fr_set_stream", "fr_sol_coords", "fr_set_state",
                 "fr_get_state", "fr_residual", "fr_rk_step", "fr_mesh_info", "fr_profile_stages",
                 "fr_mesh_geometry_host", "fr_basis_host", "fr_rk_coefficients", "fr_kinetic_energy", "fr_sgs_n_features", "fr_set_body_force",
                 "fr_batch_create", "fr_batch_create_ex", "fr_batch_step", "fr_batch_set_stream", "fr_batch_destroy",
                 "fr_set_tiles", "fr_get_tiles", "fr_tiles_in_force", "fr_autotune", "fr_set_fusion", "fr_get_fusion",
                 "fr_sgs_features", "fr_set_eddy_viscosity", "fr_set_sgs_model", "fr_get_eddy_viscosity",
                 "fr_mlp_create", "fr_mlp_destroy", "fr_mlp_set_stream", "fr_mlp_set_params",
                 "fr_mlp_get_params", "fr_mlp_get_bf16", "fr_mlp_forward", "fr_mlp_loss_grad",
                 "fr_mlp_train_step", "fr_mlp_train_step_noalloc", "fr_part_create", "fr_part_destroy", "fr_part_host",
                 "fr_part_get_mesh", "fr_part_elements", "fr_part_set_stream", "fr_halo_size", "fr_halo_pack",
                 "fr_halo_unpack", "fr_part_residual", "fr_part_rk_step"):
        getattr(L, name).restype = ctypes.c_int
    _lib = L
    return L


def _check(rc: int):
    if rc != FR_OK:
        raise FRError(rc, load().fr_last_error().decode())


def _device_ptr(t, shape, dtype, device=None, what="tensor"):
    """data_ptr() of a device tensor after checking that it is exactly what the C call reads or
    writes (a contiguous array of `shape` and `dtype` on the handle's GPU); raises before any
    library call otherwise."""
    if not getattr(t, "is_cuda", False):
        raise ValueError(f"{what}: expected a device tensor")
    if t.dtype != dtype:
        raise TypeError(f"{what}: dtype {t.dtype}, expected {dtype}")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{what}: shape {tuple(t.shape)}, expected {tuple(shape)}")
    if not t.is_contiguous():
        raise ValueError(f"{what}: must be contiguous")
    if device is not None and t.device.index != device:
        raise ValueError(f"{what}: on device {t.device.index}, the handle lives on device {device}")
    return ctypes.c_void_p(t.data_ptr())


def _current_stream():
    import torch

    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


VISCOUS = {"br2": 0, "ldg": 1}


def _desc(mesh, p, mu, gamma, prandtl, eta, flux, prec, check_finite, keep, ref=(1.0, 0.0), viscous="br2",
          ldg_tau=0.1, bc_tag=None, wall_T=1.0):
    ev = np.ascontiguousarray(mesh.elem_vert, dtype=np.int64)
    nodes = np.ascontiguousarray(mesh.elem_nodes, dtype=np.float64)
    keep.extend([ev, nodes])
    tags = None
    if bc_tag is not None:
        tags = np.ascontiguousarray(bc_tag, dtype=np.int32)
        assert tags.shape == (ev.shape[0], 6)
        keep.append(tags)
    return fr_mesh_desc(p=int(p), q=int(mesh.q), n_elem=int(ev.shape[0]), elem_vert=ev.ctypes.data,
                        elem_nodes=nodes.ctypes.data, gamma=gamma, prandtl=prandtl, mu=mu,
                        br2_eta=eta, flux=FLUX[flux], prec=PREC[prec],
                        check_finite=int(bool(check_finite)), viscous=VISCOUS[viscous],
                        ref_rho=float(ref[0]), ref_p=float(ref[1]), ldg_tau=float(ldg_tau),
                        bc_tag=tags.ctypes.data if tags is not None else None, wall_T=float(wall_T))


def rk_coefficients(scheme: str):
    """The library's RK tables (fr_rk_coefficients): (a, b) numpy arrays of the scheme's stages."""
    a, b, n = np.zeros(8), np.zeros(8), ctypes.c_int32()
    _check(load().fr_rk_coefficients(SCHEME[scheme], a.ctypes.data, b.ctypes.data, ctypes.byref(n)))
    return a[:n.value].copy(), b[:n.value].copy()


def partition_host(mesh, p: int, part, q: int, bc_tag=None):
    """Host-only split of part q (fr_part_host): (n_local, n_ghost, n_send[n_part], n_recv[n_part])."""
    keep = []
    d = _desc(mesh, p, 0.0, 1.4, 0.72, 6.0, "rusanov", "fp64", False, keep, bc_tag=bc_tag)
    part = np.ascontiguousarray(part, dtype=np.int32)
    n_part = int(part.max()) + 1
    nl, ng = ctypes.c_int64(), ctypes.c_int64()
    ns, nr = np.zeros(n_part, dtype=np.int64), np.zeros(n_part, dtype=np.int64)
    _check(load().fr_part_host(ctypes.byref(d), part.ctypes.data, n_part, int(q), ctypes.byref(nl), ctypes.byref(ng),
                               ns.ctypes.data, nr.ctypes.data))
    return nl.value, ng.value, ns, nr


def geometry_host(mesh, p: int, eta: float = 6.0, bc_tag=None):
    """Host-only mesh setup (fr_mesh_geometry_host): geo, fgeo, ftab, conn, xyz as numpy arrays."""
    keep = []
    d = _desc(mesh, p, 0.0, 1.4, 0.72, eta, "rusanov", "fp64", False, keep, bc_tag=bc_tag)
    E, Ns, Nfp = d.n_elem, (p + 1) ** 3, (p + 1) ** 2
    F = 3 * E + (int(np.sum(np.asarray(bc_tag) == 1)) // 2 if bc_tag is not None else 0)
    geo = np.empty((E, 10, Ns))
    fgeo = np.empty((F, 4, Nfp))
    ftab = np.empty((F, 4), dtype=np.int32)
    conn = np.empty((E, 6, 2), dtype=np.int32)
    xyz = np.empty((E, 3, Ns))
    _check(load().fr_mesh_geometry_host(ctypes.byref(d), geo.ctypes.data, fgeo.ctypes.data,
                                        ftab.ctypes.data, conn.ctypes.data, xyz.ctypes.data))
    return geo, fgeo, ftab, conn, xyz


def basis_host(p: int) -> dict:
    """The library's 1-D operator tables of degree p (fr_basis_host)."""
    n = p + 1
    out = {"D": np.empty((n, n)), "lm": np.empty(n), "lp": np.empty(n), "gcL": np.empty(n), "gcR": np.empty(n)}
    _check(load().fr_basis_host(int(p), *(out[k].ctypes.data for k in ("D", "lm", "lp", "gcL", "gcR"))))
    return out


class FRMesh:
    """One mesh on the current GPU (see fr_mesh_create)."""

    def __init__(self, mesh, p: int, *, mu: float = 0.0, gamma: float = 1.4, prandtl: float = 0.72,
                 eta: float = 6.0, flux: str = "rusanov", prec: str = "fp64", check_finite: bool = False,
                 stream=None, ref_rho: float = 1.0, ref_p: float = 0.0, viscous: str = "br2",
                 ldg_tau: float = 0.1, bc_tag=None, wall_T: float = 1.0):
        L = load()
        self.p = int(p)
        self.Ns = (self.p + 1) ** 3
        self.E = int(mesh.elem_vert.shape[0])
        keep = []
        d = _desc(mesh, p, mu, gamma, prandtl, eta, flux, prec, check_finite, keep, (ref_rho, ref_p), viscous,
                  ldg_tau, bc_tag, wall_T)
        self._stream = _current_stream() if stream is None else ctypes.c_void_p(stream)
        import torch

        self.device = torch.cuda.current_device()
        h = ctypes.c_void_p()
        _check(L.fr_mesh_create(ctypes.byref(d), self._stream, ctypes.byref(h)))
        self.h = h

    @classmethod
    def _part_view(cls, h, p: int, n_local: int, device: int, stream, group):
        """A part of a PartitionGroup: the group owns the handle (close() only forgets it)."""
        self = cls.__new__(cls)
        self.p = int(p)
        self.Ns = (self.p + 1) ** 3
        self.E = int(n_local)
        self.device = device
        self._stream = stream
        self._group = group
        self.h = h
        return self

    def close(self):
        if getattr(self, "_group", None) is not None:
            self.h = None
            return
        if getattr(self, "h", None) and self.h.value:
            load().fr_mesh_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def set_stream(self, stream):
        self._stream = ctypes.c_void_p(stream)
        _check(load().fr_set_stream(self.h, self._stream))

    @property
    def shape(self):
        return (self.E, 5, self.Ns)

    def sol_coords(self) -> np.ndarray:
        X = np.empty((self.E, 3, self.Ns))
        _check(load().fr_sol_coords(self.h, X.ctypes.data))
        return X

    def set_state(self, U):
        if hasattr(U, "data_ptr"):  # torch tensor on the device
            import torch

            ptr = _device_ptr(U, self.shape, torch.float64, self.device, "set_state")
            _check(load().fr_set_state(self.h, ptr, 1))
        else:
            U = np.ascontiguousarray(U, dtype=np.float64)
            assert U.shape == self.shape
            _check(load().fr_set_state(self.h, U.ctypes.data, 0))

    def get_state(self, out=None):
        if out is not None:
            import torch

            ptr = _device_ptr(out, self.shape, torch.float64, self.device, "get_state(out)")
            _check(load().fr_get_state(self.h, ptr, 1))
            return out
        U = np.empty(self.shape)
        _check(load().fr_get_state(self.h, U.ctypes.data, 0))
        return U

    def residual(self, out=None):
        """dU/dt of the current state: into a device tensor `out`, else returned as numpy."""
        if out is not None:
            import torch

            ptr = _device_ptr(out, self.shape, torch.float64, self.device, "residual(out)")
            _check(load().fr_residual(self.h, ptr, 1))
            return out
        R = np.empty(self.shape)
        _check(load().fr_residual(self.h, R.ctypes.data, 0))
        return R

    def rk_step(self, dt: float, scheme: str = "lsrk45", n_steps: int = 1):
        _check(load().fr_rk_step(self.h, float(dt), SCHEME[scheme], int(n_steps)))

    def profile_stages(self, dt: float, scheme: str = "lsrk45", n_steps: int = 1):
        """Mean kernel durations in ms from HIP events (fr_profile_stages): a dict with
        'prepass' (per launch), 'face' (per stage), 'volume_pre' (the volume kernel that also
        runs the next stage's pre-pass, per launch; 0 if none ran) and 'volume' (the volume
        kernel alone, per launch)."""
        ms = np.zeros(4)
        _check(load().fr_profile_stages(self.h, float(dt), SCHEME[scheme], int(n_steps), ms.ctypes.data))
        return dict(zip(("prepass", "face", "volume_pre", "volume"), (float(x) for x in ms)))

    def kinetic_energy(self):
        """(E_k, dE_k/dt) of the current state, volume averaged (fr_kinetic_energy)."""
        out = np.zeros(2)
        _check(load().fr_kinetic_energy(self.h, out.ctypes.data))
        return float(out[0]), float(out[1])

    def set_tiles(self, epb: int, fbs: int):
        _check(load().fr_set_tiles(self.h, int(epb), int(fbs)))

    def tiles(self):
        e, f = ctypes.c_int32(), ctypes.c_int32()
        _check(load().fr_get_tiles(self.h, ctypes.byref(e), ctypes.byref(f)))
        return e.value, f.value

    def tiles_in_force(self):
        """The tiles this mesh's own stages are launched with: tiles() once chosen, until then by size."""
        e, f = ctypes.c_int32(), ctypes.c_int32()
        _check(load().fr_tiles_in_force(self.h, ctypes.byref(e), ctypes.byref(f)))
        return e.value, f.value

    def autotune(self, n_trials: int = 3):
        """Time the tile choices with and without the fused pre-pass (fr_autotune); returns
        ((epb, fbs) chosen, ms per choice), ms[fuse * 6 + epb * 3 + fbs] (fusion() tells which
        was kept; the FP32 form's fused entries are 0)."""
        ms = np.zeros(12)
        _check(load().fr_autotune(self.h, int(n_trials), ms.ctypes.data))
        return self.tiles(), ms

    def set_fusion(self, on: bool):
        """FP64 path: each stage's volume kernel also runs the next stage's pre-pass (default)."""
        _check(load().fr_set_fusion(self.h, 1 if on else 0))

    def fusion(self) -> bool:
        v = ctypes.c_int32()
        _check(load().fr_get_fusion(self.h, ctypes.byref(v)))
        return bool(v.value)

    def set_body_force(self, g):
        """Constant body force per unit mass (3 values; None or zeros switch it off)."""
        if g is None:
            _check(load().fr_set_body_force(self.h, None))
            return
        g = np.ascontiguousarray(g, dtype=np.float64)
        assert g.shape == (3,)
        _check(load().fr_set_body_force(self.h, g.ctypes.data))

    # ---- learned eddy-viscosity closure ----
    @property
    def n_features(self) -> int:
        return self.Ns + 4

    def sgs_features(self, out=None):
        """Closure inputs of the current state (fr_sgs_features) into a float32 device tensor
        [E][Ns + 4] (allocated with torch if `out` is None)."""
        import torch

        if out is None:
            out = torch.empty((self.E, self.n_features), dtype=torch.float32, device=f"cuda:{self.device}")
        ptr = _device_ptr(out, (self.E, self.n_features), torch.float32, self.device, "sgs_features(out)")
        _check(load().fr_sgs_features(self.h, ptr))
        return out

    def set_eddy_viscosity(self, nu, prandtl_t: float = 0.9):
        """Fixed per-element nu_t [E] (numpy, or a float64 device tensor), or None to switch off."""
        if nu is None:
            _check(load().fr_set_eddy_viscosity(self.h, None, 0, prandtl_t))
        elif hasattr(nu, "data_ptr"):
            import torch

            ptr = _device_ptr(nu, (self.E,), torch.float64, self.device, "set_eddy_viscosity")
            _check(load().fr_set_eddy_viscosity(self.h, ptr, 1, prandtl_t))
        else:
            nu = np.ascontiguousarray(nu, dtype=np.float64)
            assert nu.shape == (self.E,)
            _check(load().fr_set_eddy_viscosity(self.h, nu.ctypes.data, 0, prandtl_t))

    def set_sgs_model(self, model, nu_scale: float = 0.0, prandtl_t: float = 0.9):
        """Attach an MLP (nu_t = nu_scale * model(features) per stage), or None to detach."""
        self._model = model  # kept alive while attached
        _check(load().fr_set_sgs_model(self.h, model.h if model is not None else None, float(nu_scale),
                                       float(prandtl_t)))

    def eddy_viscosity(self) -> np.ndarray:
        nu = np.empty(self.E)
        _check(load().fr_get_eddy_viscosity(self.h, nu.ctypes.data))
        return nu

    def info(self):
        E, ns, b = ctypes.c_int64(), ctypes.c_int32(), ctypes.c_int64()
        _check(load().fr_mesh_info(self.h, ctypes.byref(E), ctypes.byref(ns), ctypes.byref(b)))
        return {"n_elem": E.value, "n_sol": ns.value, "device_bytes": b.value}


H = 64
MLP_NOALLOC_MAX_N = 8192  # FR_MLP_NOALLOC_MAX_N of include/fr.h


def mlp_n_params(n_in: int) -> int:
    return int(load().fr_mlp_n_params(int(n_in)))


class MLP:
    """The closure network on the current GPU (fr_mlp_*). Parameters are float32 numpy arrays in
    the layout W1[64][n_in], b1[64], W2[64][64], b2[64], w3[64], b3[1]; inputs and targets are
    float32 device tensors."""

    def __init__(self, n_in: int, params, mean, std, stream=None):
        L = load()
        self.n_in = int(n_in)
        params = np.ascontiguousarray(params, dtype=np.float32)
        mean = np.ascontiguousarray(mean, dtype=np.float32)
        std = np.ascontiguousarray(std, dtype=np.float32)
        assert params.shape == (mlp_n_params(n_in),) and mean.shape == (n_in,) and std.shape == (n_in,)
        self._stream = _current_stream() if stream is None else ctypes.c_void_p(stream)
        h = ctypes.c_void_p()
        _check(L.fr_mlp_create(self.n_in, params.ctypes.data, mean.ctypes.data, std.ctypes.data, self._stream,
                               ctypes.byref(h)))
        self.h = h
        self.n_params = params.size

    def close(self):
        if getattr(self, "h", None) and self.h.value:
            load().fr_mlp_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def set_params(self, params):
        params = np.ascontiguousarray(params, dtype=np.float32)
        assert params.shape == (self.n_params,)
        _check(load().fr_mlp_set_params(self.h, params.ctypes.data))

    def get_params(self) -> np.ndarray:
        out = np.empty(self.n_params, dtype=np.float32)
        _check(load().fr_mlp_get_params(self.h, out.ctypes.data))
        return out

    def get_bf16(self):
        W1 = np.empty((H, self.n_in), dtype=np.uint16)
        W2 = np.empty((H, H), dtype=np.uint16)
        w3 = np.empty(H, dtype=np.uint16)
        _check(load().fr_mlp_get_bf16(self.h, W1.ctypes.data, W2.ctypes.data, w3.ctypes.data))
        return W1, W2, w3

    def _x(self, X):
        import torch

        if not getattr(X, "is_cuda", False) or X.dtype != torch.float32 or X.dim() != 2:
            raise TypeError("X: expected a 2-D float32 device tensor")
        if X.stride(1) != 1 or X.shape[1] < self.n_in or (X.shape[0] > 1 and X.stride(0) < self.n_in):
            raise ValueError("X: rows of at least n_in contiguous float32 values expected")
        return ctypes.c_void_p(X.data_ptr()), int(X.shape[0]), int(X.stride(0))

    def _t(self, t, n, what="t", at_least=False):
        """pointer of a contiguous float32 device vector of n values (at least n: an output the
        call writes n values into)"""
        import torch

        if getattr(t, "is_cuda", False) and t.is_contiguous():
            t = t.reshape(-1)
            if at_least and t.numel() >= n:
                t = t[:n] if n > 0 else t
                return _device_ptr(t, (t.numel(),), torch.float32, None, what)
        return _device_ptr(t, (n,), torch.float32, None, what)

    def forward(self, X, out=None):
        import torch

        xp, n, ld = self._x(X)
        if out is None:
            out = torch.empty(n, dtype=torch.float32, device=X.device)
        _check(load().fr_mlp_forward(self.h, xp, n, ld, self._t(out, n, "out", at_least=True)))
        return out

    def loss_grad(self, X, t):
        """(loss, gradient [n_params] float32 numpy) without updating."""
        xp, n, ld = self._x(X)
        tp = self._t(t, n)
        g = np.empty(self.n_params, dtype=np.float32)
        loss = ctypes.c_double()
        _check(load().fr_mlp_loss_grad(self.h, xp, n, ld, tp, g.ctypes.data, ctypes.byref(loss)))
        return loss.value, g

    def train_step(self, X, t, lr: float, loss_out=None):
        """One Adam step; loss_out (float32 device tensor of one element) receives the loss."""
        xp, n, ld = self._x(X)
        tp = self._t(t, n)
        lp = self._t(loss_out, 1, "loss_out") if loss_out is not None else None
        _check(load().fr_mlp_train_step(self.h, xp, n, ld, tp, float(lr), lp))

    def train_step_noalloc(self, X, t, lr: float, loss_out=None):
        """One Adam step like train_step, through fr_mlp_train_step_noalloc: its training buffers
        are the library's fixed per-GPU scratch array (nothing is allocated); n must be at most
        MLP_NOALLOC_MAX_N. Calls on one GPU share that array, so they must not overlap in time."""
        xp, n, ld = self._x(X)
        tp = self._t(t, n)
        lp = self._t(loss_out, 1, "loss_out") if loss_out is not None else None
        _check(load().fr_mlp_train_step_noalloc(self.h, xp, n, ld, tp, float(lr), lp))


class PartitionGroup:
    """A mesh split into parts by an element -> part map, advanced together on one GPU with one
    face exchange per stage (fr_part_*). parts[q] is an FRMesh view of part q (its state is
    [n_local][5][N_s] over elements[q], the part's global element indices)."""

    def __init__(self, mesh, p: int, part, *, mu: float = 0.0, gamma: float = 1.4, prandtl: float = 0.72,
                 eta: float = 6.0, flux: str = "rusanov", prec: str = "fp64", stream=None, ref_rho: float = 1.0,
                 ref_p: float = 0.0, bc_tag=None, wall_T: float = 1.0):
        import torch

        L = load()
        part = np.ascontiguousarray(part, dtype=np.int32)
        E = int(mesh.elem_vert.shape[0])
        assert part.shape == (E,)
        self.n_part = int(part.max()) + 1
        self.p = int(p)
        self.E = E
        keep = []
        d = _desc(mesh, p, mu, gamma, prandtl, eta, flux, prec, False, keep, (ref_rho, ref_p), "br2", 0.1,
                  bc_tag, wall_T)
        self._stream = _current_stream() if stream is None else ctypes.c_void_p(stream)
        self.device = torch.cuda.current_device()
        h = ctypes.c_void_p()
        _check(L.fr_part_create(ctypes.byref(d), part.ctypes.data, self.n_part, self._stream, ctypes.byref(h)))
        self.h = h
        self.parts, self.elements = [], []
        for q in range(self.n_part):
            mh, n = ctypes.c_void_p(), ctypes.c_int64()
            _check(L.fr_part_get_mesh(self.h, q, ctypes.byref(mh)))
            _check(L.fr_part_elements(self.h, q, ctypes.byref(n), None))
            ids = np.empty(n.value, dtype=np.int64)
            _check(L.fr_part_elements(self.h, q, ctypes.byref(n), ids.ctypes.data))
            self.elements.append(ids)
            self.parts.append(FRMesh._part_view(mh, p, n.value, self.device, self._stream, self))

    @property
    def shape(self):
        return (self.E, 5, (self.p + 1) ** 3)

    def set_state(self, U):
        """The whole mesh's state [E][5][N_s] (numpy), split over the parts."""
        U = np.ascontiguousarray(U, dtype=np.float64)
        assert U.shape == self.shape
        for m, ids in zip(self.parts, self.elements):
            m.set_state(U[ids])

    def get_state(self) -> np.ndarray:
        U = np.empty(self.shape)
        for m, ids in zip(self.parts, self.elements):
            U[ids] = m.get_state()
        return U

    def residual(self) -> np.ndarray:
        """The whole mesh's residual assembled from the parts' (fr_part_residual)."""
        Rs = [np.empty(m.shape) for m in self.parts]
        ptrs = (ctypes.c_void_p * self.n_part)(*[r.ctypes.data for r in Rs])
        _check(load().fr_part_residual(self.h, ctypes.cast(ptrs, ctypes.c_void_p), 0))
        R = np.empty(self.shape)
        for r, ids in zip(Rs, self.elements):
            R[ids] = r
        return R

    def rk_step(self, dt: float, scheme: str = "lsrk45", n_steps: int = 1):
        _check(load().fr_part_rk_step(self.h, float(dt), SCHEME[scheme], int(n_steps)))

    def halo_size(self, q: int, r: int):
        """(faces, bytes) of the message part q sends to part r."""
        n, b = ctypes.c_int64(), ctypes.c_int64()
        _check(load().fr_halo_size(self.parts[q].h, int(r), ctypes.byref(n), ctypes.byref(b)))
        return n.value, b.value

    def _msg(self, buf, nbytes, what):
        if not getattr(buf, "is_cuda", False) or not buf.is_contiguous():
            raise ValueError(f"{what}: expected a contiguous device tensor")
        if buf.device.index != self.device or buf.numel() * buf.element_size() < nbytes:
            raise ValueError(f"{what}: needs {nbytes} bytes on device {self.device}")
        return ctypes.c_void_p(buf.data_ptr())

    def halo_pack(self, q: int, r: int, out):
        """Part q's side of the faces it shares with part r into the device tensor out."""
        ptr = self._msg(out, self.halo_size(q, r)[1], "halo_pack")
        _check(load().fr_halo_pack(self.parts[q].h, int(r), ptr))

    def halo_unpack(self, q: int, r: int, msg):
        """The message part r packed for part q into q's ghost slots."""
        ptr = self._msg(msg, self.halo_size(r, q)[1], "halo_unpack")
        _check(load().fr_halo_unpack(self.parts[q].h, int(r), ptr))

    def close(self):
        for m in getattr(self, "parts", []):
            m.h = None
        if getattr(self, "h", None) and self.h.value:
            load().fr_part_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


BATCH_MULTI = 1  # FR_BATCH_MULTI


class Batch:
    """Meshes advanced together by one captured HIP graph per RK step (fr_batch_*). multi=True
    (the default) steps the viscous FP32-form meshes with the multi-mesh kernels, one launch per
    kernel, stage and degree; multi=False gives every mesh a graph branch of its own."""

    def __init__(self, meshes, dts, scheme: str = "lsrk45", stream=None, multi: bool = True):
        L = load()
        self.meshes = list(meshes)  # kept alive with the batch
        n = len(self.meshes)
        handles = (ctypes.c_void_p * n)(*[m.h.value for m in self.meshes])
        dt = np.ascontiguousarray(np.broadcast_to(np.asarray(dts, dtype=np.float64), (n,)))
        self._stream = _current_stream() if stream is None else ctypes.c_void_p(stream)
        h = ctypes.c_void_p()
        _check(L.fr_batch_create_ex(ctypes.cast(handles, ctypes.c_void_p), n, dt.ctypes.data, SCHEME[scheme],
                                    self._stream, BATCH_MULTI if multi else 0, ctypes.byref(h)))
        self.h = h

    def step(self, n_steps: int = 1):
        """n_steps RK steps: replays of the captured 8-step graph, then of the one-step graph."""
        _check(load().fr_batch_step(self.h, int(n_steps)))

    def close(self):
        if getattr(self, "h", None) and self.h.value:
            load().fr_batch_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass
