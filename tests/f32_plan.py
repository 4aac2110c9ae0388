"""Plan of the exact fp32 search's matrix-core filter (f32_filter_plan of the library), and searches whose workspace can
be read afterwards."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

from paper_2110_08919_amd import build as lpq_build

FIELDS = ("use", "half", "wq_half", "qtiles", "qtiles_half", "S2", "Cs", "nq_pad", "off_hard", "off_again", "off_cbuf", "off_ccnt", "off_over",
          "total")


@functools.lru_cache(None)
def _lib():
    if not os.path.exists(lpq_build.LIB):
        lpq_build.build()
    tmp = tempfile.mkdtemp()
    src, so = os.path.join(tmp, "plan.hip"), os.path.join(tmp, "libplan.so")
    with open(src, "w") as f:
        f.write('#include "lpq_internal.h"\nextern "C" void f32_plan(int64_t n, int64_t nq, int d, int k, int64_t *out) {\n'
                "const lpq::F32Filter p = lpq::f32_filter_plan(n, nq, d, k);\nint i = 0;\n"
                + "".join(f"out[i++] = (int64_t)p.{name};\n" for name in FIELDS) + "}\n")
    subprocess.run([lpq_build.HIPCC, *lpq_build.FLAGS, "-shared", src, "-o", so, "-L", lpq_build.HERE, "-l:liblpq.so",
                    f"-Wl,-rpath,{lpq_build.HERE}"], check=True)
    return C.CDLL(so)


def plan(n, nq, d, k):
    out = (C.c_int64 * len(FIELDS))()
    _lib().f32_plan(C.c_int64(n), C.c_int64(nq), d, k, out)
    return dict(zip(FIELDS, out))


def search(x, q, k, metric):
    """(ids, distances) of lpq.search_f32, the plan, and the filter's workspace as int32 words."""
    import torch
    from paper_2110_08919_amd import lpq
    (n, d), nq = x.shape, q.shape[0]
    p = plan(n, nq, d, k)
    need = lpq.lib().lpq_search_f32_workspace_bytes(n, nq, d, k) - 256
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    ids = torch.empty((nq, k), dtype=torch.int32, device="cuda")
    dists = torch.empty((nq, k), dtype=torch.float32, device="cuda")
    lpq._check(lpq.lib().lpq_search_f32(x.data_ptr(), n, x.stride(0), q.data_ptr(), nq, q.stride(0), d, k, lpq.METRIC[metric],
                                        ids.data_ptr(), dists.data_ptr(), ws.data_ptr(), need, lpq._stream()))
    torch.cuda.synchronize()
    return (ids, dists), p, ws[need - p["total"]:].view(torch.int32)


def words(p, ws, name, count):
    """`count` words of the workspace from offset `name` of the plan on."""
    at = p[name] // 4
    return ws[at:at + count]


def best_ms(fn):
    """Shortest of six calls."""
    import torch
    times = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)
