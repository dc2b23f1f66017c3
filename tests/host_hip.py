"""The library's own host code (cd_api.hip and the launchers of cd_kernels.hip) linked with
the host-only HIP runtime of host_hip.cpp: what a call allocates, launches and returns, on a
machine without a GPU. No kernel runs and no pointer that is passed in is followed."""
import ctypes as C
import importlib.util
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_17701_amd", "csrc")
PTR = {n: 0x100000000 * (i + 1) for i, n in enumerate(  # far apart: no two operands overlap
    ("x", "W_gate", "W_up", "W_down", "A_t", "B_t", "theta", "y", "h_in", "h_out", "thld", "q"))}


def build(out_dir):
    """Path of the host build in out_dir."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc missing")
    objs = []
    for src in (os.path.join(CSRC, "cd_api.hip"), os.path.join(CSRC, "cd_kernels.hip"),
                os.path.join(ROOT, "tests", "host_hip.cpp")):
        obj = os.path.join(out_dir, os.path.basename(src) + ".o")
        subprocess.run([hipcc, "--offload-host-only", "--offload-arch=gfx950", "-O0", "-std=c++17",
                        "-fPIC", "-c", "-I", os.path.join(ROOT, "include"), src, "-o", obj],
                       check=True, capture_output=True)
        objs.append(obj)
    # the device code images the objects refer to: there are none here
    und = subprocess.run(["nm", "-u", *objs], check=True, capture_output=True, text=True).stdout
    defs = sorted({w for w in und.split() if w.startswith("__hip_fatbin")})
    lib = os.path.join(out_dir, "libcountdown_host.so")
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *[f"-Wl,--defsym={d}=0" for d in defs],
                    *objs, "-lpthread", "-o", lib], check=True, capture_output=True)
    return lib


class Host:
    def __init__(self, path):
        spec = importlib.util.spec_from_file_location(
            "countdown_host_binding", os.path.join(ROOT, "paper_2505_17701_amd", "binding.py"))
        self.cd = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.cd)
        self.lib = self.cd.load_library(path)
        self.lib.host_hip_set_malloc_limit.argtypes = [C.c_size_t]
        self.lib.host_hip_live_allocations.restype = C.c_long
        self.lib.host_hip_launches.restype = C.c_char_p

    def limit(self, size=None):
        """Allocations larger than size bytes fail (None: none does)."""
        self.lib.host_hip_set_malloc_limit(C.c_size_t(-1).value if size is None else size)

    def plan(self, d_model, d_ff, max_batch=1, d_rank=0, flags=0):
        """(status, handle)"""
        h = C.c_void_p()
        return self.lib.countdown_plan_create(d_model, d_ff, max_batch, d_rank, flags,
                                              C.byref(h)), h

    def ffn(self, h, variant, B, thld=1.0):
        p, lib, cd = PTR, self.lib, self.cd
        mats = (p["W_gate"], p["W_up"], p["W_down"])
        if variant == "mono":
            return lib.countdown_ffn_mono(h, p["x"], B, *mats, thld, p["y"], None)
        if variant == "cats":
            return lib.countdown_ffn_cats(h, p["x"], B, *mats, thld, p["y"], None)
        if variant == "dense":
            return lib.countdown_ffn_dense(h, p["x"], B, *mats, p["y"], None)
        if variant == "dual_tern":
            return lib.countdown_ffn_tern(h, p["x"], B, *mats, p["theta"], thld, p["y"], None)
        pred = variant == "dual_pred"
        return lib.countdown_ffn_dual(h, p["x"], B, *mats, p["A_t"] if pred else None,
                                      p["B_t"] if pred else None, thld, p["y"], None)

    def calibrate(self, h, variant, T, k=0.9):
        p, lib, cd = PTR, self.lib, self.cd
        out = (k, p["thld"], p["q"], None)
        if variant == "dual_tern":
            return lib.countdown_calibrate_tern(h, p["x"], T, p["theta"], *out)
        v = {"mono": 0, "dual_ideal": 1, "dual_pred": 2, "cats": 4}[variant]
        pred = variant == "dual_pred"
        return lib.countdown_calibrate(h, v, p["x"], T, p["W_gate"], p["W_up"],
                                       p["A_t"] if pred else None, p["B_t"] if pred else None,
                                       *out)

    def launches(self):
        """The launches since the last call: (kernel with its template arguments, grid.x)."""
        out = [(w[0], int(w[1])) for w in
               (line.split(" ") for line in self.lib.host_hip_launches().decode().splitlines())]
        self.lib.host_hip_clear_launches()
        return out

    def ffn_topk(self, h, variant, B, k=0.9):
        p, lib = PTR, self.lib
        mats = (p["W_gate"], p["W_up"], p["W_down"])
        if variant == "dual_tern":
            return lib.countdown_ffn_tern_topk(h, p["x"], B, *mats, p["theta"], k, None, p["y"],
                                               None)
        v = {"mono": 0, "dual_ideal": 1, "dual_pred": 2, "cats": 4}[variant]
        pred = variant == "dual_pred"
        return lib.countdown_ffn_topk(h, v, p["x"], B, *mats, p["A_t"] if pred else None,
                                      p["B_t"] if pred else None, k, None, p["y"], None)

    def residual(self, h, variant, B, thld=1.0):
        p = PTR
        v = {"mono": 0, "dual_ideal": 1, "dual_pred": 2, "dense": 3, "cats": 4}[variant]
        pred = variant == "dual_pred"
        return self.lib.countdown_ffn_residual(
            h, v, p["h_in"], None, p["h_out"], 1e-5, p["x"], B, p["W_gate"], p["W_up"],
            p["W_down"], p["A_t"] if pred else None, p["B_t"] if pred else None, thld, p["y"],
            None)
