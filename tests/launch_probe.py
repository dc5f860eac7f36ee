"""What the library's set-up decides, read on the host: the coarse sweeps' launches
of a mesh, the packing of the element kernels, whether a mesh has patch records.  A few lines are
compiled with the library's host header and the packing functions of its kernel
header, and linked to it."""
import ctypes
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1506_05996_amd")

SOURCE = r"""
#include "sem_internal.h"
using namespace sem;
extern "C" int launches(const double* vtx, int64_t nv, const int64_t* hex, int64_t nh, int32_t* out, int cap) {
  HostTables T;
  build_reference(T, 2);
  build_numbering(T, hex, nh, nv);
  build_geometry(T, vtx, hex);
  build_coarse_matrices(T, vtx, hex);
  build_coarse_tree(T);
  int n = 0;
  for (int forward = 1; forward >= 0; --forward)
    for (const CoarseLaunch& L : forward ? T.fwd_launch : T.bwd_launch) {
      if (4 * n + 4 > cap) return -1;
      out[4 * n] = forward;
      out[4 * n + 1] = L.rw;
      out[4 * n + 2] = L.wide;
      out[4 * n + 3] = (int32_t)L.count;
      ++n;
    }
  return n;
}
extern "C" int has_patch_records(const double* vtx, int64_t nv, const int64_t* hex, int64_t nh, int order) {
  HostTables T;
  build_reference(T, order);
  build_numbering(T, hex, nh, nv);
  build_geometry(T, vtx, hex);
  build_patches(T, hex);
  std::vector<int32_t> pidx, pdst;
  try {
    build_patch_records(T, pidx, pdst);
  } catch (const Error&) {
    return 0;
  }
  return pidx.size() == (size_t)nh * 250 && pdst.size() == (size_t)nh * 52;
}
@PACKING@
template <int N>
static int one(int what) { return what == 0 ? line_epb<N>() : fdm_ppb<N>(); }
extern "C" int packing(int order, int what) {
  switch (order) {
    case 2: return one<2>(what);
    case 3: return one<3>(what);
    case 5: return one<5>(what);
  }
  return -1;
}
"""


def build(folder):
    with open(os.path.join(PKG, "csrc", "sem_kernels.h")) as f:
        kernels = f.read()

    def text(name):  # a packing function, from its template line to its closing brace
        at = kernels.index(f"constexpr int {name}() {{")
        return kernels[kernels.rindex("template", 0, at):kernels.index("\n}", at) + 3]

    src, lib = os.path.join(folder, "launch_probe.cpp"), os.path.join(folder, "launch_probe.so")
    with open(src, "w") as f:
        f.write(SOURCE.replace("@PACKING@", text("line_epb") + text("fdm_ppb")))
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{PKG}/csrc", src, "-o", lib, f"-L{PKG}",
                    "-l:libsem.so", f"-Wl,-rpath,{PKG}"], check=True)
    return ctypes.CDLL(lib)


def _arguments(mesh):
    vtx, hexes = np.ascontiguousarray(mesh.vtx, dtype=np.float64), np.ascontiguousarray(mesh.hex, dtype=np.int64)
    return (vtx, hexes), (vtx.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(len(vtx)),
                          hexes.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(len(hexes)))


def has_patch_records(lib, mesh, order):
    kept, args = _arguments(mesh)
    return bool(lib.has_patch_records(*args, order))


def coarse_launches(lib, mesh):
    """[(forward, rows per wave, rows beyond 128 entries, workgroups)] of one coarse solve."""
    kept, args = _arguments(mesh)
    out = np.zeros(1024, dtype=np.int32)
    n = lib.launches(*args, out.ctypes.data_as(ctypes.c_void_p), out.size)
    assert n >= 0
    return [tuple(int(v) for v in row) for row in out[:4 * n].reshape(-1, 4)]


def grid(elements, per_group):
    """Workgroups of an element kernel (whole turns over the 8 XCDs)."""
    return -(-(-(-elements // per_group)) // 8) * 8
