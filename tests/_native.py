"""Compiles and runs a C++ program against the library's internals, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1811_00156_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def build_host(tmp_path, source: str) -> str:
    """A host program that includes csrc/internal.h and links the library.  A HIP
    function that the program defines takes the runtime's place."""
    src, exe = tmp_path / "prog.cpp", tmp_path / "prog"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror=return-type", "-rdynamic", "-D__HIP_PLATFORM_AMD__",
                    f"-I{ROCM}/include", f"-I{ROOT}/include", f"-I{PKG}/csrc", str(src), "-o", str(exe), f"-L{PKG}",
                    "-l:libaiwc_rf.so", f"-Wl,-rpath,{PKG}", f"-L{ROCM}/lib", f"-Wl,-rpath,{ROCM}/lib", "-lamdhip64"],
                   check=True)
    return str(exe)


def run_exe(exe: str, args=()) -> str:
    return subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout


def run_host(tmp_path, source: str, args=()) -> str:
    return run_exe(build_host(tmp_path, source), args)
