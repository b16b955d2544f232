"""libjas as a CPU library: its HIP sources over the stand-in runtime of this
folder, under AddressSanitizer (see hip/hip_runtime.h).

build(folder) makes the library; a child process started with environment(rt)
binds it with attach(path), after which the package's bindings run on it (numpy
arrays take the place of device buffers, the null stream of torch's).
"""
import concurrent.futures as cf
import ctypes
import glob
import os
import re
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_1911_04200_amd", "csrc")


def compiler():
    """(clang++, AddressSanitizer runtime), or None where they are not installed."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cxx = os.path.join(rocm, "llvm", "bin", "clang++")
    rt = glob.glob(os.path.join(rocm, "llvm", "lib", "clang", "*", "lib", "linux", "libclang_rt.asan-x86_64.so"))
    return (cxx, rt[0]) if shutil.which(cxx) and rt else None


def rewrite(text):
    """HIP constructs a C++ compiler does not take, in the stand-in's terms."""
    # register hints
    text = re.sub(r'asm\s*(volatile)?\s*\(""\s*:\s*"\+v"\((?:[^()]|\([^()]*\))*\)\);', ";", text)
    text = re.sub(r"__attribute__\(\(amdgpu_waves_per_eu\((?:[^()]|\((?:[^()]|\([^()]*\))*\))*\)\)\)", "", text)
    text = text.replace("__attribute__((address_space(4)))", "")
    # a place in the code stands for one operation: no unrolled copies of it
    text = re.sub(r"#pragma unroll.*", "", text)
    text = re.sub(r"extern __shared__ (?:__attribute__\(\(aligned\(16\)\)\) )?([\w ]+?) (\w+)\[\];",
                  r"\1 *\2 = reinterpret_cast<\1 *>(model::dynamic_lds);", text)
    # a wave's lanes read a counter before the first of them adds to it
    text = text.replace("if (valid) b0 = wcnt[w][d];", "if (valid) b0 = wcnt[w][d]; model::exchange(0);")
    return re.sub(r"(\b[A-Za-z_]\w*(?:<[^<>;(){}]*>)?)<<<(.*?)>>>\s*\(",
                  lambda m: 'model::Launch("%s", %s)(%s, ' % (m.group(1), m.group(2), m.group(1)), text, flags=re.S)


def build(folder, csrc=CSRC, changes=()):
    """Compiles the library into folder; returns (its path, the sanitizer's runtime).
    changes: (file, text, text in its place), each found once."""
    cxx, rt = compiler()
    sources = []
    for f in sorted(os.listdir(csrc)):
        with open(os.path.join(csrc, f)) as fh:
            text = fh.read()
        for name, old, new in changes:
            if name == f:
                assert text.count(old) == 1, (f, old)
                text = text.replace(old, new)
        text = rewrite(text)
        if f == "memory.hip":  # runtime.cpp has the buffers
            text = text.replace("*cache_alloc(", "*unused_cache_alloc(").replace("void cache_free(", "void unused_cache_free(")
        name = f[:-4] + ".cpp" if f.endswith(".hip") else f
        with open(os.path.join(folder, name), "w") as fh:
            fh.write(text)
        if f.endswith(".hip"):
            sources.append(os.path.join(folder, name))
    sources.append(os.path.join(HERE, "runtime.cpp"))
    flags = ["-O1", "-g1", "-fno-unroll-loops", "-fPIC", "-std=c++17", "-w", "-fsanitize=address", "-ffp-contract=off",
             "-fno-omit-frame-pointer", "-I", HERE, "-I", folder, "-I", os.path.join(os.path.dirname(os.path.dirname(csrc)), "include")]

    def compile_one(src):
        obj = os.path.join(folder, os.path.basename(src) + ".o")
        subprocess.check_call([cxx, *flags, "-c", src, "-o", obj])
        return obj

    with cf.ThreadPoolExecutor(8) as ex:
        objs = list(ex.map(compile_one, sources))
    lib = os.path.join(folder, "libjas_model.so")
    subprocess.check_call([cxx, "-shared", "-fsanitize=address", "-shared-libasan", "-o", lib, *objs])
    return lib, rt


def environment(rt):
    return dict(os.environ, LD_PRELOAD=rt, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0:detect_odr_violation=0",
                OMP_NUM_THREADS="1", PYTHONPATH=os.pathsep.join([ROOT, HERE]))


def attach(path):
    """The package's bindings on the model; returns (bindings, library)."""
    from paper_1911_04200_amd import jas

    lib = jas.load(path)
    for name, ret, args in (("model_lazy", None, [ctypes.c_int]), ("model_drain", None, []),
                            ("model_pending", ctypes.c_long, []), ("model_fail_at", None, [ctypes.c_long]),
                            ("model_allocations", ctypes.c_long, []), ("model_live", ctypes.c_long, []),
                            ("model_atomic_adds", ctypes.c_long, []), ("model_atomic_swaps", ctypes.c_long, []),
                            ("model_barriers", ctypes.c_long, []), ("model_launches", ctypes.c_long, [ctypes.c_char_p]),
                            ("model_blocks", ctypes.c_long, [ctypes.c_char_p])):
        f = getattr(lib, name)
        f.restype, f.argtypes = ret, args
    jas._stream = lambda stream: stream if isinstance(stream, int) else None
    lib.model_fail_at(-1)
    return jas, lib
