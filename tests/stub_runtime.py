"""libgear.so over tests/stub_runtime.cpp, in a child process: what every call
would launch, on tables and batches of any size, without a GPU."""
import ctypes
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "stub_runtime.cpp")


def build(folder):
    out = os.path.join(str(folder), "libstub_runtime.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), "-o", out, SOURCE],
                   check=True)
    return out


def run(lib, module, function, *args):
    """function(Runtime, *args) of a test module in a child process; returns its (JSON) result."""
    code = "import json, sys; from tests.stub_runtime import Runtime; import %s as m; print('RESULT', json.dumps(" \
           "m.%s(Runtime(sys.argv[1]), *json.loads(sys.argv[2]))))" % (module, function)
    r = subprocess.run([sys.executable, "-c", code, lib, json.dumps(args)], cwd=ROOT, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return json.loads(r.stdout.split("RESULT ", 1)[1])


class Segment(ctypes.Structure):
    _fields_ = [("src", ctypes.c_uint64), ("dst", ctypes.c_uint64), ("bytes", ctypes.c_int64)]


class SegmentArgs(ctypes.Structure):
    _fields_ = [("task0", ctypes.c_uint32 * 40), ("seg", Segment * 40)]


class WordArgs(ctypes.Structure):
    _fields_ = [("task0", ctypes.c_uint32), ("n", ctypes.c_int32), ("dst", ctypes.c_uint64), ("at", ctypes.c_int64),
                ("N", ctypes.c_int64), ("words", ctypes.c_uint32 * 512)]


class Runtime:
    """Loads the stub before libgear.so, so that the library's HIP calls bind to
    it; `launches` holds (kernel name, grid, block, whatever `reader` makes of the
    arguments), `copies` the (dst, src, bytes) of every copy."""

    def __init__(self, path):
        self.stub = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
        from paper_2310_05205_amd import gear
        self.gear, self.lib = gear, gear.lib()
        self.launches, self.copies, self.reader = [], [], lambda name, args: None
        callback = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_uint32, ctypes.c_uint32,
                                    ctypes.POINTER(ctypes.c_void_p))
        self._launch = callback(lambda name, grid, block, args: self.launches.append(
            (name.decode(), grid, block, self.reader(name.decode(), args))))
        copy = ctypes.CFUNCTYPE(None, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint64)
        self._copy = copy(lambda *a: self.copies.append(a))
        self.stub.stub_on_launch(self._launch)
        self.stub.stub_on_copy(self._copy)
        self.stub.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
        self.stub.stub_lock.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
        self.stub.stub_locked_offset.restype = ctypes.c_uint64

    def device(self, nbytes):
        p = ctypes.c_void_p()
        self.stub.hipMalloc(ctypes.byref(p), nbytes)
        return p.value

    def table(self, elem_bytes, N, T, residency=0):
        return self.gear.gear_table_create(list(elem_bytes), N, T, residency, 0)

    def column(self, table, c):
        return self.gear.gear_table_column(table, c)[0]


class ColTask(ctypes.Structure):
    _fields_ = [("src", ctypes.c_uint64), ("out", ctypes.c_uint64), ("W", ctypes.c_int64), ("n", ctypes.c_int64),
                ("recip", ctypes.c_uint64), ("E", ctypes.c_int32), ("epw", ctypes.c_uint32),
                ("magic", ctypes.c_uint32), ("wpp", ctypes.c_uint16), ("width", ctypes.c_uint8),
                ("layout", ctypes.c_uint8), ("pad", ctypes.c_int64)]


class CollectArgs(ctypes.Structure):
    _fields_ = [("task0", ctypes.c_int32 * 16), ("idx", ctypes.c_uint64), ("start", ctypes.c_uint64),
                ("status", ctypes.c_uint64), ("N", ctypes.c_int64), ("B", ctypes.c_int32), ("T", ctypes.c_int32),
                ("L", ctypes.c_int32), ("pad", ctypes.c_int32 * 5), ("col", ColTask * 16)]


assert ctypes.sizeof(ColTask) == 64 and CollectArgs.col.offset % 64 == 0


def read_collect(name, args):
    """The arguments of collect_kernel: elements per thread, first tasks, columns."""
    if "collect_kernel" not in name:
        return None
    a = ctypes.cast(args[0], ctypes.POINTER(CollectArgs)).contents
    used = [k for k in range(16) if a.task0[k] != 0x7FFFFFFF]
    return (int(name.split("collect_kernelILi")[1][0]), [a.task0[k] for k in used],
            [{f: getattr(a.col[k], f) for f in ("out", "W", "n", "width", "layout", "wpp", "epw")} for k in used])


def read_segments(name, args):
    """The arguments of copy_segments_kernel and copy_segments_words_kernel."""
    if "copy_segments" not in name:
        return None
    a = ctypes.cast(args[0], ctypes.POINTER(SegmentArgs)).contents
    w = ctypes.cast(args[1], ctypes.POINTER(WordArgs)).contents if "words" in name else None
    return ([a.task0[k] for k in range(40)], [(g.src, g.dst, g.bytes) for g in a.seg],
            None if w is None else (w.task0, w.n, w.dst, w.at))


def segment_copies(launch):
    """The (dst, src, bytes) that the workgroups of a segment launch copy."""
    _, grid, _, (task0, seg, words) = launch
    end = grid if words is None else words[0]
    out = []
    for k, (src, dst, nbytes) in enumerate(seg):
        if task0[k] == 0xFFFFFFFF:
            break
        stop = min(task0[k + 1], end) if k + 1 < 40 else end
        out.append((dst, src, min(nbytes, (stop - task0[k]) * 1024 - dst % 16)))
    return out
