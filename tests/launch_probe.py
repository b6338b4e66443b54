"""Run in a process of its own (no torch: the recorder must be found before
the HIP runtime): reads a JSON list of [function, [arguments]] from stdin,
calls libstagefrontier with the recorder in place of the runtime and prints,
per call, its status and the launches it made.  An argument "p<i>" is the
i-th of a set of far apart, aligned addresses; nothing reads them."""
import ctypes
import json
import sys


def main():
    rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    rec.rec_name.restype = ctypes.c_char_p
    rec.rec_lds.restype = ctypes.c_uint64
    lib = ctypes.CDLL(sys.argv[2])
    out = []
    for name, args in json.load(sys.stdin):
        fn = getattr(lib, name)
        fn.restype = ctypes.c_int
        conv = []
        for a in args:
            if isinstance(a, str):
                conv.append(ctypes.c_void_p((int(a[1:]) + 1) << 52))
            else:
                kind, v = a
                conv.append(ctypes.c_int32(v) if kind == "i" else ctypes.c_int64(v))
        rec.rec_clear()
        rc = fn(*conv)
        out.append([rc, [[rec.rec_name(i).decode(), rec.rec_grid(i), rec.rec_block(i), rec.rec_lds(i)]
                         for i in range(rec.rec_launches())]])
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    main()
