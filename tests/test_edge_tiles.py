"""The tiles of host-only meshes (tests/host/edge_tiles.cpp, tile_shapes.cpp, linked
with the library; no GPU): strips, grids of many macros, fans whose centre has
64 and more copies, at the smallest levels and where the lists change kind."""
import os
import subprocess

import numpy as np

import paper_2305_15116_amd as P
from paper_2305_15116_amd import build
from paper_2305_15116_amd import workloads as W
from test_gpu_many_macros import grid2, grid3

HERE = os.path.dirname(os.path.abspath(__file__))


def fan(dim, n):
    ring = [[np.cos(2 * np.pi * i / n), np.sin(2 * np.pi * i / n), 0.5] for i in range(n)]
    if dim == 2:
        return (np.array([[0.0, 0.0]] + [r[:2] for r in ring]),
                W.shuffle_cell_orders(np.array([[0, 1 + i, 1 + (i + 1) % n] for i in range(n)]), 2))
    return (np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 1.0]] + ring),
            W.shuffle_cell_orders(np.array([[0, 1, 2 + i, 2 + (i + 1) % n] for i in range(n)]), 2))


def _run(source, tmp_path):
    P.lib()
    exe = str(tmp_path / "check")
    root = os.path.dirname(HERE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(root, "include"), "-I" + build.CSRC, os.path.join(HERE, "host", source),
                    build.LIB, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + os.path.dirname(build.LIB),
                    "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)
    meshes = [(W.unit_triangle(), 8), (W.strip_2d(7), 8), (W.strip_2d(44), 8), (grid2(16), 6), (fan(2, 6), 6), (fan(2, 64), 4),
              (fan(2, 70), 5), (W.unit_tet(), 6), (W.strip_3d(7), 5), (grid3(3), 4), (fan(3, 6), 5), (fan(3, 64), 3), (fan(3, 70), 4)]
    text = []
    for (co, ce), level in meshes:
        text.append(f"{co.shape[1]} {level} {len(co)} {len(ce)}")
        text += [" ".join(repr(float(v)) for v in co.ravel()), " ".join(str(int(v)) for v in ce.ravel())]
    r = subprocess.run([exe], input="\n".join(text), capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout


def test_every_copy_in_one_tile(tmp_path):
    _run("edge_tiles.cpp", tmp_path)


def test_tile_shapes_have_kernels(tmp_path):
    _run("tile_shapes.cpp", tmp_path)
