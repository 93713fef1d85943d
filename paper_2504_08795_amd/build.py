"""Builds libdaris.so for gfx950 with hipcc, in-tree: the device code objects (every kernel of csrc/*kernels.hip), linked
into the library as data, and the host runtime that dispatches them (HSA queues) behind the C ABI."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdaris.so")
# device source -> symbol prefix of its code object in the library
DEVICE_SOURCES = {"kernels.hip": "daris_kernels", "taps_kernels.hip": "daris_taps_kernels", "image_kernels.hip": "daris_image_kernels", "block_kernels.hip": "daris_block_kernels",
                  "point_kernels.hip": "daris_point_kernels"}
# ... of the kernels that compute several layers in a row
JOINED_SOURCES = {"joined_kernels.hip": "daris_joined_kernels", "tall_kernels.hip": "daris_tall_kernels", "pointwise_kernels.hip": "daris_pointwise_kernels"}
HOST_SOURCES = ["aql.cpp", "launch.cpp", "sched_core.cpp", "net_plan.cpp", "net_encode.cpp", "daris_api.cpp"]
COMMON = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-Wall", "-Wno-unused-function"]
# no packed fp32 arithmetic in device code (some forms have given wrong results on this hardware)
DEVICE_FLAGS = COMMON + ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "--no-gpu-bundle-output"]
HOST_FLAGS = COMMON + ["-fPIC"]

BLOB_ASM = """
    .section .rodata
    .global {name}_co
    .global {name}_co_end
    .balign 4096
{name}_co:
    .incbin "{path}"
{name}_co_end:
    .byte 0
    .section .note.GNU-stack,"",@progbits
"""


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    asm = ""
    for src, name in {**DEVICE_SOURCES, **JOINED_SOURCES}.items():
        code_object = os.path.join(CSRC, name + ".co")
        _run([hipcc] + DEVICE_FLAGS + ["-c", os.path.join(CSRC, src), "-o", code_object], verbose)
        asm += BLOB_ASM.format(name=name, path=code_object)
    blob_s = os.path.join(CSRC, "kernels_blob.S.tmp.s")
    with open(blob_s, "w") as f:
        f.write(asm)
    objs = [os.path.join(CSRC, "kernels_blob.o")]
    _run(["gcc", "-c", blob_s, "-o", objs[0]], verbose)
    os.remove(blob_s)
    # the one translation unit with both host and device code: the static scratch array and its address lookup
    obj = os.path.join(CSRC, "static_scratch.hip.o")
    _run([hipcc] + HOST_FLAGS + ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-c", os.path.join(CSRC, "static_scratch.hip"), "-o", obj], verbose)
    objs.append(obj)
    for src in HOST_SOURCES:
        obj = os.path.join(CSRC, src + ".o")
        _run([hipcc] + HOST_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj], verbose)
        objs.append(obj)
    _run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs + ["-L/opt/rocm/lib", "-lhsa-runtime64", "-lpthread", "-ldl"], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
