"""Compile the stepping kernels for the CPU (tests only), the way
build_sim.py does for the queue worker: one host thread per lane, dynamic LDS
from the emulated workgroup, waits and compiler fences as wave
reconvergence, every label, offset and edge index checked."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2602_10080_amd", "csrc")
KERNEL = os.path.join(CSRC, "mlmq_step.hip")

CHECKS = [
    ("ld_label(c.a.lab + v)", 'ld_label(c.a.lab + simt_chk(v, c.a.n, "lab", __LINE__))'),
    ("c.a.lab + (uint32_t)e[u]", 'c.a.lab + simt_chk((uint32_t)e[u], c.a.n, "lab", __LINE__)'),
    ("c.a.lab + (uint32_t)e)", 'c.a.lab + simt_chk((uint32_t)e, c.a.n, "lab", __LINE__))'),
    ("c.a.lab + gv", 'c.a.lab + simt_chk(gv, c.a.n, "lab", __LINE__)'),
    ("c.a.off[v]", 'c.a.off[simt_chk(v, c.a.n, "off", __LINE__)]'),
    ("c.a.ioff[v]", 'c.a.ioff[simt_chk(v, c.a.n, "ioff", __LINE__)]'),
    ("c.a.adj[i]", 'c.a.adj[simt_chk(i, (uint32_t)c.a.off[c.a.n], "adj", __LINE__)]'),
    ("c.a.adj[x + sub]", 'c.a.adj[simt_chk(x + sub, (uint32_t)c.a.off[c.a.n], "adj", __LINE__)]'),
    ("c.a.iadj[i]", 'c.a.iadj[simt_chk(i, (uint32_t)c.a.off[c.a.n], "iadj", __LINE__)]'),
    ("c.a.iadj[x + sub]", 'c.a.iadj[simt_chk(x + sub, (uint32_t)c.a.off[c.a.n], "iadj", __LINE__)]'),
    ("list[(uint64_t)j * cap + (idx - excl)]",
     'list[(uint64_t)simt_chk(j, 64u, "segment", __LINE__) * cap + simt_chk(idx - excl, cap, "list", __LINE__)]'),
]


def transformed_source() -> str:
    src = open(KERNEL).read()
    for a, b in CHECKS:
        assert a in src, a
        src = src.replace(a, b)
    src = src.replace("extern __shared__ uint64_t smem[];",
                      "uint64_t* smem = reinterpret_cast<uint64_t*>(simt::group->lds);")
    src = re.sub(r'asm volatile\("([^"]*)"\s*:::\s*"memory"\);', lambda mo: 'simt::wave_sync_at("asm ' + mo.group(1) + '");', src)
    cut = src.index("hipError_t launch_step_init(")
    return src[:cut] + "\n}  // namespace mlmq\n"


def build(out_dir: str) -> str:
    work = os.path.join(out_dir, "tmp%d" % os.getpid())
    os.makedirs(work, exist_ok=True)
    inc = os.path.join(work, "sim_step_kernels.inc")
    with open(inc, "w") as f:
        f.write(transformed_source())
    lib = os.path.join(out_dir, "libsimstep.so")
    tmp = os.path.join(work, os.path.basename(lib))
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-g", "-fPIC", "-shared", "-pthread", "-w", "-I", HERE, "-iquote",
                           CSRC, "-iquote", work, os.path.join(HERE, "step_harness.cpp"), "-o", tmp])
    os.replace(tmp, lib)
    os.remove(inc)
    os.rmdir(work)
    return lib


if __name__ == "__main__":
    print(build(os.path.join(ROOT, "_build", "simt")))
