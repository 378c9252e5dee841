"""Build libod.so (HIP kernels + C++ runtime + C ABI) in-tree for gfx950."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libod.so")
SOURCES = ["kernels.hip", "deep.hip", "deep2d.hip", "plan.cpp", "od_api.cpp", "od_capi.cpp", "tune.cpp", "server.cpp", "launch_bench.hip"]

# Bit-exactness: no contraction into FMA, correctly rounded fp32 division,
# subnormals kept.  Packed-fp32 instructions are disabled for the device.
DEVICE_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math",
    "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _resource_table(remarks: str) -> str:
    """Rows {"<kernel>", total SGPRs, VGPRs, LDS bytes} from the compiler's
    kernel-resource-usage remarks; kernel names demangled without their
    return type and parameter list (e.g. od::k_persistent<double, 32, 16, false>)."""
    rows, cur = {}, None
    for ln in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", ln)
        if m:
            cur = m.group(1)
            rows[cur] = {}
            continue
        m = re.search(r"remark:\s+(\w[^:]*?): (\S+) \[-Rpass", ln)
        if cur and m:
            rows[cur][m.group(1)] = m.group(2)
    names = list(rows)
    dem = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                         check=True).stdout.splitlines()
    out = ["// generated by build.py from -Rpass-analysis=kernel-resource-usage; do not edit"]
    for mangled, pretty in zip(names, dem):
        r = rows[mangled]
        key = pretty.split("(")[0]
        if key.startswith("void "):
            key = key[5:]
        out.append('{"%s", %d, %d, %d},' % (key, int(r.get("TotalSGPRs", 0)), int(r.get("VGPRs", 0)),
                                           int(r.get("LDS Size [bytes/block]", 0))))
    return "\n".join(out) + "\n"


def build(verbose: bool = False) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    cc = hipcc()
    # the kernels' register usage, read by the cooperative-launch sizing
    # (resources.cpp): a device-only compile of kernels.hip with the
    # compiler's resource remarks, run beside the other compiles
    rem_cmd = [cc, *DEVICE_FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
               os.path.join(CSRC, "kernels.hip"), "-o", os.path.join(objdir, "kernels_device_only.o")]
    rem = subprocess.Popen(rem_cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    procs, objs = [], []
    for src in SOURCES:
        obj = os.path.join(objdir, src.rsplit(".", 1)[0] + ".o")
        objs.append(obj)
        cmd = [cc, *DEVICE_FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            failed.append((src, out))
        elif verbose and out.strip():
            print(out, flush=True)
    rem_out, _ = rem.communicate()
    if rem.returncode != 0:
        failed.append(("kernels.hip (resource remarks)", rem_out))
    else:
        table = _resource_table(rem_out)
        if table.count("\n") < 20:
            failed.append(("kernels.hip (resource remarks)", "no kernel-resource-usage remarks found"))
        else:
            with open(os.path.join(objdir, "kernel_resources.inc"), "w") as f:
                f.write(table)
            obj = os.path.join(objdir, "resources.o")
            cmd = [cc, *DEVICE_FLAGS, "-I", objdir, "-x", "hip", "-c", os.path.join(CSRC, "resources.cpp"), "-o", obj]
            r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            if r.returncode != 0:
                failed.append(("resources.cpp", r.stdout))
            objs.append(obj)
    if failed:
        for src, out in failed:
            sys.stderr.write(f"--- {src} failed ---\n{out}\n")
        raise RuntimeError("libod build failed: " + ", ".join(s for s, _ in failed))
    tmp = LIB + ".tmp"
    link = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs, "-lpthread"]
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.run(link, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
