"""Which kernels a call takes, without a GPU: the host side of the C ABI linked with launchers that write down what they are asked
for (route_recorder.hip)."""
import ctypes
import os
import subprocess
import tempfile

from paper_2401_04658_amd import binding, build

HERE = os.path.dirname(os.path.abspath(__file__))
UNITS = 256   # compute units that the host side plans for where it sees no device
P = 1 << 30   # an aligned address; nothing reads it
_lib = None


def lib():
    global _lib
    if _lib is None:
        api = os.path.join(os.path.dirname(binding.lib_path()), "_build", "la2_api.o")
        if not os.path.exists(api):
            build.build()
        folder = tempfile.mkdtemp()
        obj, so = os.path.join(folder, "route_recorder.o"), os.path.join(folder, "libroutes.so")
        subprocess.check_call([build.HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-fPIC", "-Wall", "-Wno-unused-command-line-argument", "-c",
                               os.path.join(HERE, "route_recorder.hip"), "-o", obj])
        subprocess.check_call([build.HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", so, obj, api])
        _lib = ctypes.CDLL(so)
        for name in ("la2_workspace_bytes", "la2_varlen_workspace_bytes"):
            getattr(_lib, name).restype = ctypes.c_size_t
    return _lib


def desc(b, h, n, d, dtype=binding.LA2_BF16, packed=False):
    if packed:
        return binding.la2_desc(b, h, n, d, dtype, 0, 0, d, h * d)
    return binding.la2_desc(b, h, n, d, dtype, 0, h * n * d, n * d, d)


def _take():
    size = 1 << 16
    while True:
        out = ctypes.create_string_buffer(size)
        n = lib().routes_take(out, size)
        assert n >= 0
        launches = []
        for line in out.value.decode().splitlines():
            words = line.split()
            launches.append(dict((w.split("=", 1) for w in words[1:]), launcher=words[0]))
        for x in launches:
            for key, value in x.items():
                x[key] = int(value) if value.lstrip("-").isdigit() else value
        return launches


def _p(x):
    return ctypes.c_void_p(x)


def _size(x):
    return ctypes.c_size_t(x)


ADDRESS = {name: P + (i << 24) for i, name in enumerate(("q", "k", "v", "d_o", "lam", "o", "dq", "dk", "dv", "kv_init", "kv_final", "d_kv_final",
                                                          "d_kv_init", "cu", "ws", "ws_f", "rstd", "d_u"))}


def forward(d, init=None, final=None, total=None, workspace=None):
    """Launches of la2_fwd_state (total: la2_fwd_varlen_state) with a workspace as large as asked for."""
    A, L = ADDRESS, lib()
    _take()
    if total is None:
        need = L.la2_workspace_bytes(ctypes.byref(d), binding.LA2_OP_FWD_STATE) if workspace is None else workspace
        st = L.la2_fwd_state(ctypes.byref(d), _p(A["q"]), _p(A["k"]), _p(A["v"]), _p(A["lam"]), _p(init), _p(A["o"]), _p(final), _p(A["ws_f"]),
                             _size(need), _p(0))
    else:
        need = L.la2_varlen_workspace_bytes(ctypes.byref(d), ctypes.c_int64(total), binding.LA2_OP_FWD) if workspace is None else workspace
        st = L.la2_fwd_varlen_state(ctypes.byref(d), _p(A["cu"]), ctypes.c_int64(total), _p(A["q"]), _p(A["k"]), _p(A["v"]), _p(A["lam"]), _p(init),
                                    _p(A["o"]), _p(final), _p(A["ws_f"]), _size(need), _p(0))
    assert st == 0, st
    return _take()


def backward(d, init=None, d_final=None, d_init=None, total=None, saved=False, workspace=None):
    """Launches of la2_bwd_saved (total: la2_bwd_varlen_state)."""
    A, L = ADDRESS, lib()
    _take()
    front = (_p(A["q"]), _p(A["k"]), _p(A["v"]), _p(A["d_o"]), _p(A["lam"]), _p(init), _p(d_final), _p(A["dq"]), _p(A["dk"]), _p(A["dv"]), _p(d_init))
    if total is None:
        need = L.la2_workspace_bytes(ctypes.byref(d), binding.LA2_OP_BWD_STATE) if workspace is None else workspace
        f = L.la2_workspace_bytes(ctypes.byref(d), binding.LA2_OP_FWD_STATE)
        st = L.la2_bwd_saved(ctypes.byref(d), *front, _p(A["ws_f"] if saved else 0), _size(f), 0, _p(A["ws"]), _size(need), _p(0))
    else:
        need = L.la2_varlen_workspace_bytes(ctypes.byref(d), ctypes.c_int64(total), binding.LA2_OP_BWD) if workspace is None else workspace
        st = L.la2_bwd_varlen_state(ctypes.byref(d), _p(A["cu"]), ctypes.c_int64(total), *front, _p(A["ws"]), _size(need), _p(0))
    assert st == 0, st
    return _take()


def one_launch(launches):
    """The launch of all three scans of a backward pass among them, or None."""
    found = [x for x in launches if x["launcher"] in ("bwd_scans_bf16", "bwd_scans_wide")]
    assert len(found) <= 1
    return found[0] if found else None
