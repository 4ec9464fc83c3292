"""The library's kernels on the CPU: the sources compiled against tests/cpu_device (a launch runs
its workgroups one after another, with a schedule of the waves that the test chooses), and one
step of calls through the C ABI on host arrays."""
from __future__ import annotations

import dataclasses
import os
import re
import shutil
import struct
import subprocess
import tempfile

import numpy as np

from workloads import page_table
from workloads.values import host_normal_f16, q_values

HERE = os.path.dirname(os.path.abspath(__file__))
DEVICE = os.path.join(HERE, "cpu_device")
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_26666_amd", "csrc")
ROUTES = ("plan_decode", "noalloc", "fused", "separate", "rect", "buckets")
ASCENDING, DESCENDING = 0, 1  # wave schedules; any other number is the seed of a pseudo-random one


def compiler():
    for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("amdclang++"), shutil.which("clang++")):
        if c and os.path.exists(c):
            return c
    return None


def build(folder, csrc=CSRC):
    """The program of the sources in `csrc` (seconds)."""
    flags = [compiler(), "-std=c++17", "-O2", "-fno-pie", "-ffp-contract=off", "-w", "-I", DEVICE, "-I", csrc]
    with open("/proc/cpuinfo") as f:
        have = set(re.findall(r"\b(?:fma|f16c)\b", f.read()))
    flags += [f"-m{x}" for x in sorted(have)]  # else in software: the same values, much slower
    units = [(os.path.join(csrc, "pkv_kernels.hip"), "kernels"), (os.path.join(csrc, "pkv_capi.cpp"), "capi"),
             (os.path.join(DEVICE, "emu.cpp"), "emu"), (os.path.join(DEVICE, "main.cpp"), "main")]
    objs, jobs = [], []
    for src, name in units:
        objs.append(os.path.join(folder, name + ".o"))
        jobs.append(subprocess.Popen([*flags, "-x", "c++", "-c", src, "-o", objs[-1]], stderr=subprocess.PIPE, text=True))
    for j in jobs:
        err = j.communicate()[1]
        assert j.returncode == 0, err
    exe = os.path.join(folder, "cpu_device")
    subprocess.run([compiler(), "-no-pie", *objs, "-o", exe], check=True)
    return exe


class Program:
    def __init__(self, exe):
        self.exe = exe
        names = subprocess.run(["nm", "-C", exe], capture_output=True, text=True, check=True).stdout
        self.names = {int(a, 16): n for a, n in re.findall(r"^([0-9a-f]+) [tTwW] (.*)$", names, flags=re.M)}

    def kernel(self, at):
        """`stream_kernel<4, 8, true, false>` of a launch's address."""
        m = re.search(r"(\w+_kernel(?:<[^()]*>)?)", self.names.get(at, ""))
        return m.group(1) if m else hex(at)


@dataclasses.dataclass
class Answer:
    status: int
    error_bits: int
    counters_left: int  # completion counters that are not zero
    num_tasks: int
    out: np.ndarray     # fp16 [B, hq, 128]
    offsets: np.ndarray
    tasks: np.ndarray   # [max_tasks, 5]


class Call:
    """Inputs of calls on one workspace; lens may be [calls, B]."""

    def __init__(self, lens, hq=32, hkv=8, seed=0):
        r = np.random.Generator(np.random.PCG64(seed))
        self.lens = np.atleast_2d(np.asarray(lens, dtype=np.int32))
        self.B, self.hq, self.hkv = self.lens.shape[1], hq, hkv
        self.bt, self.num_pages = page_table(np.maximum(self.lens.max(axis=0), 1), 16, 0.3, r)
        self.bt = np.ascontiguousarray(self.bt, dtype=np.int32)
        shape = (int(self.num_pages), 16, hkv, 128)
        self.k, self.v = host_normal_f16(shape, r), host_normal_f16(shape, r)
        self.q = q_values(self.B, hq, 128, r)

    def run(self, program, route, params, *, order=ASCENDING, compute_units=2, S=0, row_ids=(), bucket_tokens=0,
            sm_scale=1.0, given=None, num_tasks=None, max_tasks=None):
        """([Answer per call], [(kernel, grid) of the first call])."""
        page_size, tile, hkv, smin, smax, target, policy = params
        if max_tasks is None:
            max_tasks = self.B * self.hkv * max(smax, S)
        words = [ROUTES.index(route), order, compute_units, len(self.lens), self.B, self.hq, self.hkv, int(self.num_pages),
                 self.bt.shape[1], max_tasks, S, len(row_ids), bucket_tokens, -1 if given is None else len(given[0]),
                 0 if given is None else (len(given[0]) if num_tasks is None else num_tasks)]
        data = struct.pack("<15if7i", *words, sm_scale, *params)
        parts = [self.q, self.k, self.v, self.bt, self.lens, np.asarray(row_ids, dtype=np.int32)]
        if given is not None:
            parts += [np.asarray(given[0], dtype=np.int32), np.asarray(given[1], dtype=np.int32)]
        with tempfile.TemporaryDirectory() as d:
            req, ans = os.path.join(d, "req"), os.path.join(d, "ans")
            with open(req, "wb") as f:
                f.write(data)
                for p in parts:
                    f.write(np.ascontiguousarray(p).tobytes())
            p = subprocess.run([program.exe, req, ans], capture_output=True, text=True, timeout=300)
            assert p.returncode == 0, (p.returncode, p.stderr)
            raw = open(ans, "rb").read()
        answers, at = [], 0

        def take(dtype, shape):
            nonlocal at
            n = int(np.prod(shape)) * np.dtype(dtype).itemsize
            a = np.frombuffer(raw[at:at + n], dtype=dtype).reshape(shape)
            at += n
            return a

        for _ in self.lens:
            head = take(np.int32, (4,)).tolist()
            out = take(np.float16, (self.B, self.hq, 128))
            answers.append(Answer(*head, out, take(np.int32, (self.B + 1,)), take(np.int32, (max_tasks, 5))))
        launched = [(program.kernel(int(a, 16)), int(g)) for a, g in re.findall(r"^([0-9a-f]+) (\d+)$", p.stdout, flags=re.M)]
        return answers, launched
