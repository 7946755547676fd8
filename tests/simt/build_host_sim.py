"""Compile the library's host code for the CPU (tests only), over the
stand-in device of host/device.cpp."""
import glob
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2602_10080_amd", "csrc")
HOST = os.path.join(HERE, "host")


def build(out_dir: str) -> str:
    work = os.path.join(out_dir, "host%d" % os.getpid())
    os.makedirs(work, exist_ok=True)
    lib = os.path.join(out_dir, "libsimhost.so")

    def one(src):
        obj = os.path.join(work, os.path.basename(src) + ".o")
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-pthread", "-w", "-I", HOST, "-iquote", CSRC,
                               "-c", src, "-o", obj])
        return obj

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(one, sorted(glob.glob(os.path.join(CSRC, "*.cpp"))) + [os.path.join(HOST, "device.cpp")]))
    tmp = os.path.join(work, "lib.so")
    subprocess.check_call(["g++", "-shared", "-pthread", *objs, "-o", tmp])
    os.replace(tmp, lib)
    for o in objs:
        os.remove(o)
    os.rmdir(work)
    return lib


if __name__ == "__main__":
    print(build(os.path.join(ROOT, "_build", "simt")))
