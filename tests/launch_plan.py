"""What a Log-Int-Softmax call would launch, without a GPU: the C ABI's host code
and the launch selection (csrc/lis_dispatch.h) linked against stand-ins for the
launchers (abi_launch_stubs.cpp)."""
import collections
import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2111_13824_amd", "csrc")
Plan = collections.namedtuple("Plan", "kernel nc dt half waves split blocks lds fp gathered")
KERNELS = ("unit", "tile", "stream")


class Launches:
    def __init__(self, folder):
        so = os.path.join(str(folder), "libfqvit_plan.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(CSRC, "fqvit_abi.cpp"),
                        os.path.join(HERE, "abi_launch_stubs.cpp"), "-o", so], check=True)
        from paper_2111_13824_amd import binding
        self.lib = binding.load(so)

    def _last(self, status):
        assert status == 0, status
        v = (ctypes.c_longlong * 10)()
        self.lib.fq_test_last_plan(v)
        return Plan(KERNELS[v[0]], v[1], v[2], bool(v[3]), v[4], v[5], v[6], v[7], bool(v[8]), v[9])

    def head(self, G, Lq, Lk, d, s=2.0 ** -10, bits=4, exp_n=20, Hb=0, codes_out=False):
        """The launch of lis_attention_head on 16-byte aligned tensors."""
        p = 4096
        return self._last(self.lib.lis_attention_head(
            p, p if Hb else None, Hb, G, Lq, Lk, s, bits, exp_n, p, 0, d, p,
            p if codes_out else None, (Lk + 1) // 2 if codes_out else 0, None))

    def codes(self, G, Lq, Lk, s=2.0 ** -10, bits=4, exp_n=20, pad=0):
        """The launch of lis_softmax_log4, code rows padded by `pad` bytes."""
        p = 4096
        ld = ((Lk + 1) // 2 if bits <= 4 else Lk) + pad
        return self._last(self.lib.lis_softmax_log4(p, G, Lq, Lk, None, 0, s, bits, exp_n, p, ld, None))
