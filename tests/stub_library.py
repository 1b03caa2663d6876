"""The package over a build of the library for the host only, linked with the stand-in HIP runtime of
hip_stub_runtime.cpp: every call works without a GPU, no kernel runs, and the names of the kernels that a
call enqueues can be read back."""
import ctypes
import importlib.util
import math
import os
import re
import subprocess
import sys

from conftest import ROOT

PACKAGE = os.path.join(ROOT, "paper_1606_07676_amd")
CLANGXX = "/opt/rocm/llvm/bin/clang++"


def compile_host(directory, sources):
    """(source, is HIP) -> object files for the host only"""
    objs = []
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PACKAGE, "csrc")]
    common = ["-O3", "-std=c++17", "-fPIC"]
    for src, hip in sources:
        obj = os.path.join(directory, os.path.basename(src) + ".o")
        if hip:
            cmd = ["hipcc", "-x", "hip", "--cuda-host-only", "-fuse-cuid=none", *common, *inc, "-c", src, "-o", obj]
        else:
            cmd = [CLANGXX, *common, *inc, "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-c", src, "-o", obj]
        proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert proc.returncode == 0, proc.stdout[-3000:]
        objs.append(obj)
    return objs


PLAN, RUNTIME = os.path.join(PACKAGE, "csrc", "iso_plan.cpp"), os.path.join(ROOT, "tests", "hip_stub_runtime.cpp")


def build(directory):
    objs = compile_host(directory, [(os.path.join(PACKAGE, "csrc", "iso_api.hip"), True), (PLAN, False), (RUNTIME, False)])
    lib = os.path.join(directory, "libiso_on_stub.so")
    subprocess.run([CLANGXX, "-shared", "-Wl,-Bsymbolic", *objs, "-o", lib], check=True)
    return lib


def build_driver(directory, source):
    """An executable from a test driver that includes the library's host code."""
    objs = compile_host(directory, [(os.path.join(ROOT, "tests", source), True), (PLAN, False), (RUNTIME, False)])
    exe = os.path.join(directory, os.path.splitext(source)[0])
    subprocess.run([CLANGXX, *objs, "-o", exe], check=True)
    return exe


class StubLibrary:
    """`iso`: the package, bound to the stub build."""

    def __init__(self, directory):
        path = build(directory)
        spec = importlib.util.spec_from_file_location("iso_on_stub", os.path.join(PACKAGE, "__init__.py"),
                                                      submodule_search_locations=[PACKAGE])
        self.iso = importlib.util.module_from_spec(spec)
        sys.modules["iso_on_stub"] = self.iso
        spec.loader.exec_module(self.iso)
        sys.modules["iso_on_stub.binding"]._LIB_PATH = path
        self.lib = ctypes.CDLL(path)
        self.lib.stub_device_alloc.restype = ctypes.c_void_p
        self.lib.stub_device_alloc.argtypes = [ctypes.c_size_t]
        self.lib.stub_device_free.argtypes = [ctypes.c_void_p]
        self.lib.stub_log_size.restype = ctypes.c_long
        self.lib.stub_log_grid.restype = ctypes.c_long
        self.lib.stub_log_grid.argtypes = [ctypes.c_long]
        self.lib.stub_log_name.restype = ctypes.c_char_p
        self.lib.stub_log_name.argtypes = [ctypes.c_long]
        self.iso.load_library()

    def comm(self, dims, offsets, periodic=None):
        if periodic is None:
            return self.iso.iso_neighborhood_create(dims, offsets)
        return self.iso.iso_neighborhood_create_mesh(dims, periodic, offsets)

    def launched(self, call):
        """The kernels that call() enqueues, as name<template arguments>; the vector types are called v8 and v16."""
        self.lib.stub_log_clear()
        call()
        names = [self.lib.stub_log_name(i).decode() for i in range(self.lib.stub_log_size())]
        self.grids = [self.lib.stub_log_grid(i) for i in range(len(names))]      # workgroups of these launches
        if not names:
            return []
        out = subprocess.run(["c++filt"], input="\n".join(names), stdout=subprocess.PIPE, text=True, check=True).stdout
        out = out.replace("unsigned int __vector(4)", "v16").replace("unsigned int __vector(2)", "v8")
        return [re.sub(r"^void |iso::|\([^()]*\)$", "", n) for n in out.split("\n") if n]

    def buffers(self, *sizes):
        """Context manager: one 'device' buffer per size (None for 0)."""
        return _Buffers(self.lib, sizes)

    def request(self, comm, dims, s, op, alg, m, layout, bufs):
        iso = self.iso
        init = iso.iso_neighbor_alltoall_init_layout if op == iso.ISO_OP_ALLTOALL else iso.iso_neighbor_allgather_init_layout
        send, recv, work = bufs
        return init(send, recv, m, layout, work, comm, alg, workspace_bytes=iso.iso_workspace_bytes(comm, op, alg, m))

    def start(self, dims, offsets, op, alg, m, layout=0, periodic=None, by_rounds=False):
        """The kernels of one iso_start of a request over equal blocks (by_rounds: of its whole launch list)."""
        iso, p, s = self.iso, math.prod(dims), len(offsets)
        comm = self.comm(dims, offsets, periodic)
        with self.buffers(p * m * (s if op == iso.ISO_OP_ALLTOALL else 1), p * s * m,
                          iso.iso_workspace_bytes(comm, op, alg, m)) as bufs:
            req = self.request(comm, dims, s, op, alg, m, layout, bufs)
            n = iso.iso_request_info(req)["launches"]
            out = self.launched(lambda: iso.iso_start_range(req, 0, n, 0) if by_rounds else iso.iso_start(req, 0))
            iso.iso_request_free(req)
        return out

    def start_unequal(self, dims, offsets, alg, sizes, periodic=None):
        """The kernels of one iso_start of an all-to-all over blocks of `sizes` bytes, packed rows."""
        iso, p = self.iso, math.prod(dims)
        comm = self.comm(dims, offsets, periodic)
        displs, row = [sum(sizes[:i]) for i in range(len(sizes))], sum(sizes)
        wsb = iso.iso_workspace_bytes_v(comm, iso.ISO_OP_ALLTOALL, alg, sizes)
        with self.buffers(p * row, p * row, wsb) as (send, recv, work):
            req = iso.iso_neighbor_alltoallv_init(send, sizes, displs, row, recv, sizes, displs, row, work, comm, alg,
                                                  workspace_bytes=wsb)
            out = self.launched(lambda: iso.iso_start(req, 0))
            iso.iso_request_free(req)
        return out


class _Buffers:
    def __init__(self, lib, sizes):
        self._lib, self._sizes = lib, sizes

    def __enter__(self):
        self._ptrs = [self._lib.stub_device_alloc(n) if n else None for n in self._sizes]
        return self._ptrs

    def __exit__(self, *exc):
        for q in self._ptrs:
            if q:
                self._lib.stub_device_free(q)
