"""Builds tests/frame_harness.cpp against the library and calls it."""
import ctypes as C
import os
import subprocess

from paper_2008_06134_amd import vi

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2008_06134_amd", "csrc")
_lib = None


def lib():
    global _lib
    if _lib is None:
        out, src = os.path.join(ROOT, "_build", "frame_harness.so"), os.path.join(HERE, "frame_harness.cpp")
        os.makedirs(os.path.dirname(out), exist_ok=True)
        newer = [src, os.path.join(CSRC, "vi_internal.h"), os.path.join(ROOT, "include", "vi.h"), vi.LIB_PATH]
        if not os.path.exists(out) or any(os.path.getmtime(out) <= os.path.getmtime(f) for f in newer):
            subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                                   "-I", "/opt/rocm/include", src, vi.LIB_PATH,
                                   f"-Wl,-rpath,{os.path.dirname(vi.LIB_PATH)}", "-o", out])
        vi.lib()
        _lib = C.CDLL(out)
        args = [C.POINTER(vi.Volume_t), C.POINTER(vi.TF_t), C.POINTER(vi.Slices_t), C.POINTER(vi.Camera_t), C.c_int,
                C.c_float, C.POINTER(vi.RenderOpts_t), C.c_void_p]
        _lib.h_window.argtypes = args
        _lib.h_render.argtypes = args + [C.c_void_p, C.c_int]
    return _lib


def _args(vol, tf, stack, cam, mode, step, opts, out):
    return (C.byref(vol), C.byref(tf), C.byref(stack), C.byref(vi.camera(cam)), vi.MODES[mode], step,
            C.byref(vi.render_opts(opts)), out)


def window(vol, tf, stack, cam, mode, step, opts=None):
    """(fits, staged) for structures whose pointers need not be real (host only)."""
    r = lib().h_window(*_args(vol, tf, stack, cam, mode, step, opts, 1 << 20))
    assert r >= 0, vi.lib().vi_last_error().decode()
    return bool(r & 1), bool(r & 2)


def render(vol, tf, stack, cam, mode, step, opts, stage):
    """The image with the window on or off."""
    import torch
    img = torch.empty(cam["height"], cam["width"], 4, device=vol.data.device)
    rc = lib().h_render(*_args(vol.s, tf.s, stack.s, cam, mode, step, opts, img.data_ptr()),
                        torch.cuda.current_stream().cuda_stream, int(stage))
    assert rc == 0, (rc, vi.lib().vi_last_error().decode())
    return img
