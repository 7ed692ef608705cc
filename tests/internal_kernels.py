"""The library's internal launchers for tests of single kernels (ctypes on their C++ symbols; not part of the C ABI):
the wide update from FP16 pairs and the symmetric factorization, on FP32 systems in device memory."""
import ctypes

import numpy as np
import torch

from paper_2311_12134_amd._lib import lib

NB, PERM_STRIDE = 64, 2 + 4 * 64
JOB = np.dtype([(f, np.int64) for f in ("a_off", "v_off", "x_off", "r_off", "piv_off", "liz_off")] +
               [(f, np.int32) for f in ("atom", "energy", "nl", "n", "npad", "info", "ld", "pad")])
_F2 = "15HIP_vector_typeIfLj2EE"


class Scratch(ctypes.Structure):
    _fields_ = [("p", ctypes.c_void_p), ("bytes", ctypes.c_size_t)]


def piv_ints(npad):
    return npad + npad // NB * PERM_STRIDE


class Systems:
    """FP32 copies of square complex matrices whose sizes are multiples of 64, with their descriptors."""

    def __init__(self, mats):
        self.mats = mats
        self.npad = [len(m) for m in mats]
        assert all(n % NB == 0 for n in self.npad)
        jobs = np.zeros(len(mats), JOB)
        jobs["a_off"] = np.concatenate([[0], np.cumsum([n * n for n in self.npad])[:-1]])
        jobs["piv_off"] = np.concatenate([[0], np.cumsum([piv_ints(n) for n in self.npad])[:-1]])
        jobs["n"] = jobs["npad"] = self.npad
        self.jobs = torch.from_numpy(jobs.view(np.uint8).reshape(-1).copy()).cuda()
        self.work = torch.from_numpy(np.concatenate([m.astype(np.complex64).reshape(-1) for m in mats])).cuda()
        self.piv = torch.zeros(sum(piv_ints(n) for n in self.npad), dtype=torch.int32, device="cuda")
        self.info = torch.zeros(len(mats), dtype=torch.int32, device="cuda")

    def results(self):
        torch.cuda.synchronize()
        flat, out, o = self.work.cpu().numpy(), [], 0
        for n in self.npad:
            out.append(flat[o:o + n * n].reshape(n, n))
            o += n * n
        return out


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def pair_scratch(rows, cols, kd, jobs):
    """Scratch of the pair update for that many jobs at a time."""
    size = lib()._ZN4lsms15half2_job_bytesEiii
    size.restype = ctypes.c_size_t
    return torch.zeros(jobs * size(rows, cols, kd), dtype=torch.uint8, device="cuda")


def pair_update(s, kd, jobs_at_once=None, c_begin=None, c_end=0, lower=False):
    """A22 -= L21 U12 of the first kd columns and rows, by the FP16-pair kernels."""
    n = max(s.npad)
    cb = kd if c_begin is None else c_begin
    rows, cols = n - kd, (min(c_end, n) if c_end else n) - cb
    buf = pair_scratch(rows, cols, kd, jobs_at_once or len(s.mats))
    call = lib()["_ZN4lsms17launch_gemm_half2EPKNS_7JobDescEiiiiiiiiP%sRKNS_12Half2ScratchEP12ihipStream_tb" % _F2]
    call.restype = None
    call(_ptr(s.jobs), len(s.mats), rows, cols, 0, kd, kd, cb, c_end, _ptr(s.work),
         ctypes.byref(Scratch(buf.data_ptr(), buf.numel())), _stream(), ctypes.c_bool(lower))
    torch.cuda.synchronize()


def fp32_update(s, kd, tiling=2):
    """The same by an FP32 matrix-core tiling."""
    n = max(s.npad)
    call = lib()["_ZN4lsms19launch_gemm_f32_anyEiPKNS_7JobDescEiiiiiiiiP%sRKNS_12Half2ScratchEP12ihipStream_t" % _F2]
    call.restype = None
    call(tiling, _ptr(s.jobs), len(s.mats), n - kd, n - kd, 0, kd, kd, kd, 0, _ptr(s.work),
         ctypes.byref(Scratch(None, 0)), _stream())
    torch.cuda.synchronize()


def ldlt(s, tall_rows):
    """The symmetric factorization; panels of at most tall_rows rows by the panel kernel as a whole."""
    size = lib()._ZN4lsms18ldlt_scratch_bytesEi
    size.restype = ctypes.c_size_t
    buf = torch.zeros(size(len(s.mats)), dtype=torch.uint8, device="cuda")
    call = lib()["_ZN4lsms15ldlt_factor_f32EPKNS_7JobDescEiiP%sPiS6_P12ihipStream_tPNS_12GemmProfilerERKNS_12Half2ScratchEiPv"
                 % _F2]
    call.restype = None
    call(_ptr(s.jobs), len(s.mats), max(s.npad), _ptr(s.work), _ptr(s.piv), _ptr(s.info), _stream(), None,
         ctypes.byref(Scratch(None, 0)), tall_rows, _ptr(buf))
    torch.cuda.synchronize()
