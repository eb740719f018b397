"""Which kernels a call of the C ABI launches, without a GPU: a child process loads a stand-in for the HIP runtime
(tests/host_hip/recorder.c) ahead of the library, makes the calls with stand-in pointers and reports every launch."""
import ctypes
import json
import os
import re
import subprocess
import sys
from pathlib import Path

HERE = Path(__file__).resolve().parent
LIB = HERE.parent / "paper_2403_07221_amd" / "liblookupffn.so"
FAKE = 1 << 24          # aligned stand-in for a device pointer
MODES = {"plain": 0, "weighted": 1, "probes": 2}

# p pointer, q 64-bit count, i int
SIGNATURES = {
    "lookupffn_gather": "pppqiiiipqp", "lookupffn_gather_weighted": "ppppqiiiipqp", "lookupffn_gather_probes": "ppppqiiiipqp",
    "lookupffn_hash": "pppqiiiiip", "lookupffn_hash_weighted": "ppppqiiiiip", "lookupffn_hash_probes": "ppppqiiiiip",
    "lookupffn_hash_bh": "pppqiiiiiipqp", "lookupffn_hash_bh_weighted": "ppppqiiiiiipqp",
    "lookupffn_forward": "ppppqiiiiiiipqp", "lookupffn_forward_weighted": "ppppqiiiiiiipqp", "lookupffn_forward_probes": "ppppqiiiiiiipqp",
    "lookupffn_forward_bh": "ppppqiiiiiiiipqp", "lookupffn_forward_bh_weighted": "ppppqiiiiiiiipqp",
    "lookupffn_set_option": "si",
}
CTYPES = {"p": ctypes.c_void_p, "q": ctypes.c_int64, "i": ctypes.c_int, "s": ctypes.c_char_p}

_i, _q, _p = ctypes.c_int, ctypes.c_longlong, ctypes.c_void_p


class GatherLdsArgs(ctypes.Structure):  # csrc/gather_lds_kernel.hpp
    _fields_ = [("packed", _p), ("wpk", _p), ("n_pad", _q), ("tables", _p), ("y", _p), ("y_kind", _i), ("n", _q), ("k", _i),
                ("tau", _i), ("d_out", _i), ("nvec", _i), ("n_slices", _i), ("token_splits", _i), ("n_units", _i),
                ("blocks_per_xcd", _i), ("unit_chunks", _i)]


class Launch:
    def __init__(self, line):
        symbol, x, y, z, block, lds, raw = line.split()
        self.grid, self.block, self.lds = (int(x), int(y), int(z)), int(block), int(lds)
        name = re.search(r"lffn\d+(\w+?_kernel)(?:I(.*?)EEv)?", symbol)
        self.kernel = name.group(1)
        self.params = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", (name.group(2) or "") + "E"))
        self.raw = bytes.fromhex(raw)

    def args(self, struct):
        return struct.from_buffer_copy(self.raw)

    def pointers(self, count):
        return tuple(int.from_bytes(self.raw[8 * i:8 * i + 8], "little") for i in range(count))

    def __repr__(self):
        return f"{self.kernel}{list(self.params)} grid {self.grid} block {self.block} lds {self.lds}"


def build(tmp):
    so = Path(tmp) / "recorder.so"
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), str(HERE / "host_hip" / "recorder.c")], check=True)
    return so


def record(recorder, calls, compute_units=256, lib=LIB):
    """The launches of each call (name, *args); set_option calls take effect for those after them."""
    job = json.dumps([str(recorder), str(lib), compute_units, calls])
    out = subprocess.run([sys.executable, str(HERE / "recorded.py")], input=job, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-2000:]
    result = []
    for status, text in json.loads(out.stdout):
        assert status == 0, f"{calls[len(result)]}: status {status}"
        result.append([Launch(line) for line in text.splitlines()])
    return result


def gather(mode, n, k, tau, d_out, table_dtype=0):
    pointers = [FAKE] * (3 if mode == "plain" else 4)
    name = "lookupffn_gather" + ("" if mode == "plain" else "_" + mode)
    return [name, *pointers, n, k, tau, d_out, table_dtype, None, 0, None]


def option(key, value):
    return ["lookupffn_set_option", key, value]


def main():
    recorder, lib, compute_units, calls = json.load(sys.stdin)
    R = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)
    R.recorder_take.restype = ctypes.c_char_p
    R.recorder_set_compute_units(compute_units)
    L = ctypes.CDLL(lib, mode=os.RTLD_NOW)
    out = []
    for name, *args in calls:
        f = getattr(L, name)
        f.argtypes = [CTYPES[c] for c in SIGNATURES[name]]
        status = f(*[a.encode() if isinstance(a, str) else a for a in args])
        out.append((status, R.recorder_take().decode()))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    main()
