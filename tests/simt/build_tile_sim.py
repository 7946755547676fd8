"""Compile the tiled solve's kernels for the CPU (tests only), as
build_step_sim.py does for the stepping ones."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2602_10080_amd", "csrc")
KERNEL = os.path.join(CSRC, "mlmq_tile.hip")

CHECKS = [
    ("l.lab + v)", 'l.lab + simt_chk(v, S, "label", __LINE__))'),
    ("l.lab + u0,", 'l.lab + simt_chk(u0, S, "label", __LINE__),'),
    ("l.lab + u,", 'l.lab + simt_chk(u, S, "label", __LINE__),'),
    ("l.extra[k]", 'l.extra[simt_chk(k, nx, "extra", __LINE__)]'),
    ("l.extra[i] = ", 'l.extra[simt_chk(i, a.g.xcap, "extra", __LINE__)] = '),
    ("a.lab[dst]", 'a.lab[simt_chk(dst, (uint64_t)a.g.tiles << a.g.sbits, "id", __LINE__)]'),
    ("l.ctl[kCtlMine + r / gridDim.x]", 'l.ctl[kCtlMine + simt_chk(r / gridDim.x, kTileVisits, "visit", __LINE__)]'),
]


def transformed_source() -> str:
    src = open(KERNEL).read()
    for a, b in CHECKS:
        assert a in src, a
        src = src.replace(a, b)
    src = src.replace("extern __shared__ uint64_t smem[];",
                      "uint64_t* smem = reinterpret_cast<uint64_t*>(simt::group->lds);")
    src = re.sub(r'asm volatile\("([^"]*)"\s*:::\s*"memory"\);', lambda mo: 'simt::wave_sync_at("asm ' + mo.group(1) + '");', src)
    a, b = src.index("hipError_t tile_set_lds("), src.index("size_t tile_lds_bytes(")
    cut = min(a, b)
    sizes = src[b:src.index("}", b) + 2]
    return src[:cut] + sizes + "\n}  // namespace mlmq\n"


def build(out_dir: str) -> str:
    work = os.path.join(out_dir, "tmp%d" % os.getpid())
    os.makedirs(work, exist_ok=True)
    inc = os.path.join(work, "sim_tile_kernels.inc")
    with open(inc, "w") as f:
        f.write(transformed_source())
    lib = os.path.join(out_dir, "libsimtile.so")
    tmp = os.path.join(work, os.path.basename(lib))
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-g", "-fPIC", "-shared", "-pthread", "-w", "-I", HERE, "-iquote",
                           CSRC, "-iquote", work, os.path.join(HERE, "tile_harness.cpp"), "-o", tmp])
    os.replace(tmp, lib)
    os.remove(inc)
    os.rmdir(work)
    return lib


if __name__ == "__main__":
    print(build(os.path.join(ROOT, "_build", "simt")))
