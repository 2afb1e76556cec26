"""Drives libpolymul.so on a HIP runtime without a GPU (host/fake_hip.cpp) and prints what the
library asked of it.  Run as a program of its own: argv[1] the runtime, argv[2] the library, argv[3]
the binding's source, argv[4] a list of calls as JSON; prints one JSON result per call."""
import ctypes
import importlib.util
import json
import sys

vp = ctypes.c_void_p


def main():
    fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
    fake.fake_hip_log.restype = ctypes.c_char_p
    fake.fake_hip_reset.argtypes = [ctypes.c_uint64]
    fake.fake_hip_peak.restype = fake.fake_hip_used.restype = ctypes.c_uint64
    lib = ctypes.CDLL(sys.argv[2])
    spec = importlib.util.spec_from_file_location("binding", sys.argv[3])
    binding = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(binding)
    for name, (res, args) in binding._SIGNATURES.items():
        if hasattr(lib, name):
            getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
    held = []

    def value(x):
        if isinstance(x, dict) and "u32" in x:
            held.append((ctypes.c_uint32 * len(x["u32"]))(*x["u32"]))
            return ctypes.cast(held[-1], vp)
        if isinstance(x, dict) and "out" in x:
            held.append(ctypes.c_uint64() if x["out"] == 64 else ctypes.c_uint32())
            return ctypes.byref(held[-1])
        return x

    for call in json.loads(sys.argv[4]):
        fake.fake_hip_reset(call.get("limit", (1 << 64) - 1))
        before = fake.fake_hip_used()
        if "plan" in call:  # groups [n, q, count]; arrays at made-up addresses
            arr = (binding._Group * len(call["plan"]))()
            at = 1 << 40
            for i, (n, q, count) in enumerate(call["plan"]):
                size = 4 * n * count
                arr[i] = binding._Group(at, at + size, at + 2 * size, n, q, count, 4)
                at += 3 * size
            h = vp()
            st = lib.polymul_plan_create(ctypes.byref(h), ctypes.cast(arr, vp), len(call["plan"]), 1)
            held_bytes = fake.fake_hip_used() - before
            if st == 0:
                st = lib.polymul_plan_execute(h, None)
                lib.polymul_plan_destroy(h)
            out = {"held": held_bytes}
        else:
            st = getattr(lib, call["fn"])(*[value(x) for x in call["args"]])
            out = {"out": [int(x.value) for x in held if hasattr(x, "value")]}
            held.clear()
        out.update(status=st, leaked=fake.fake_hip_used() - before, peak=fake.fake_hip_peak() - before,
                   launches=[line.split(" ") for line in fake.fake_hip_log().decode().splitlines()])
        print(json.dumps(out))


if __name__ == "__main__":
    main()
