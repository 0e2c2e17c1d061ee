"""The bounds of the spike lists that pass through LDS in pieces, on the CPU:
the address of a list's end stays within the piece, however many groups of
four before it the list ended."""
import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_ends_of_lists_stay_within_the_piece(tmp_path):
    so = str(tmp_path / "gather_host.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-nogpulib",
                    os.path.join(HERE, "gather_host.hip"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.gather_piece_end.restype = ctypes.c_uint
    cap, e8 = lib.gather_cap(), lib.gather_entries()
    for base in (e8, e8 + 64):
        # the wrap came where base + 8 end went below zero
        for end in (-2**27, -10**6, -base // 8 - 1, -base // 8, -base // 8 + 1, -cap, -1, 0, 1, cap - 1, cap, cap + 1, 2**27):
            assert lib.gather_piece_end(base, end) == base + 8 * min(max(end, 0), cap), end
