"""Compile the HIP library in-tree for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(PKG, "csrc", "nbos_replay.hip")
LIB = os.path.join(PKG, "libnbos.so")
PROFILE_LIB = os.path.join(PKG, "libnbos_pathprofile.so")      # diagnostic build, see path_profile.py

HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               # all lanes take part in every LDS atomic (one instruction, no branch): without this the optimiser wraps the
               # sums that several lanes bring to one counter in reductions over the wave (measured without it: 64 hosts
               # 68.0 -> 74.7 ms, 30 hosts 28.0 -> 31.3, 24 hosts 47.3 -> 54.5, 300 short replays 0.84 -> 0.95)
               "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
               # a replay is one long dependent chain run by a lone wave: schedule for instruction-level
               # parallelism, not for occupancy (measured: c4 239 -> 230 ms, c3 101 -> 98.8 ms, c2 37.4 -> 36.9 ms)
               "-mllvm", "-amdgpu-sched-strategy=iterative-ilp",
               # almost all control flow is wave-uniform: leave regions without a divergent branch as they are written
               # (by default they are rebuilt too, with a flag in a scalar register pair for every join; measured:
               # 30 hosts 37.5 -> 35.7 ms, 64 hosts 94.3 -> 89.6 ms, closed loops 78.8 -> 74.3 and 194.6 -> 188.2 ms)
               "-mllvm", "-structurizecfg-skip-uniform-regions=1",
               # a block that is only reached by a branch begins on a 64-byte line: a lone wave waits for every fetch
               # (measured: 64 hosts 70.2 -> 68.0 ms, 30 hosts 28.5 -> 28.0, closed loops 57.8 -> 55.5 and 131.1 -> 128.8,
               # 768 hosts 167.6 -> 166.1; Batch 151.7 -> 152.6; 32 and 128 bytes: the same)
               "-mllvm", "-align-all-nofallthru-blocks=6"]


def _hipcc(out: str, extra: list[str], verbose: bool) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra, "-o", out, SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print(" ".join(cmd))
    return out


def build_library(verbose: bool = False) -> str:
    """The product library."""
    return _hipcc(LIB, [], verbose)


def build_profile_library(verbose: bool = False) -> str:
    """The same sources with the path profile compiled in (-DNBOS_PATH_PROFILE): a diagnostic build that
    only `python -m paper_2503_20591_amd.path_profile` loads."""
    return _hipcc(PROFILE_LIB, ["-DNBOS_PATH_PROFILE"], verbose)


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_profile_library(verbose=True))
