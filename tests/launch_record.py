"""The host side of the library with its launches recorded instead of made: which kernels a call would launch and with
what arguments, on the CPU.  relay_attn.hip is compiled with the launchers below in place of the kernel files."""
import ctypes
import functools
import hashlib
import json
import os
import subprocess
import tempfile

import paper_2402_14808_amd as ra
from paper_2402_14808_amd import binding, build

LAUNCHERS = r"""
#include "ra_kernels.h"
#include <cstdio>
#include <string>
static std::string log_;
static void add(const char *name, std::initializer_list<std::pair<const char *, long long>> fields,
                const char *list = nullptr, const int *values = nullptr, int n = 0) {
    log_ += std::string(log_.empty() ? "" : ",") + "{\"launch\":\"" + name + "\"";
    for (const auto &f : fields) log_ += std::string(",\"") + f.first + "\":" + std::to_string(f.second);
    if (list) {
        log_ += std::string(",\"") + list + "\":[";
        for (int i = 0; i < n; ++i) log_ += (i ? "," : "") + std::to_string(values[i]);
        log_ += "]";
    }
    log_ += "}";
}
extern "C" const char *take_launches() {
    static std::string out;
    out = "[" + log_ + "]";
    log_.clear();
    return out.c_str();
}
namespace ra {
hipError_t launch_decode_direct(const DirectArgs &a, const DirectOne *, const DirectMany *, int, hipStream_t) {
    return add("direct", {{"tokens", a.n_tokens}, {"append", a.k_new != nullptr}}), hipSuccess;
}
hipError_t launch_relay_tiles(const TileArgs &a, int, hipStream_t) {
    return add("tiles", {{"sys_items", a.n_sys_items}, {"ctx_waves", a.ctx_waves}, {"floor", a.ctx_t_floor},
                         {"slots", a.n_ctx_slots}, {"chunk", a.sys_chunk}, {"sys_chunks", a.n_sys_chunks},
                         {"light", a.ctx_light_waves}, {"rows_sys", a.n_sys_rowblocks > 0},
                         {"append", a.k_new != nullptr}}), hipSuccess;
}
hipError_t launch_relay_rows(const RowsArgs &a, int, hipStream_t) {
    return add("rows", {{"whole", a.whole}, {"chunk", a.sys_chunk}, {"part", a.ctx_part}, {"sys_items", a.n_sys_items}},
               "prompts", a.pfx_len, a.n_prefixes > 1 ? a.n_prefixes : 0), hipSuccess;
}
hipError_t launch_fuse(const FuseArgs &a, int, hipStream_t) {
    return add("fuse", {{"rows", a.rows}, {"partials", a.n_partials}, {"likely", a.n_likely}}), hipSuccess;
}
hipError_t launch_ctx_decode(const CtxArgs &, int, int, hipStream_t) { return add("naive", {}), hipSuccess; }
hipError_t launch_cache_append(const AppendArgs &, hipStream_t) { return add("append", {}), hipSuccess; }
hipError_t launch_system_fill(const SysFillArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_validate(const ValidateArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_probe(const void *, size_t, int, void *, hipStream_t) { return hipSuccess; }
hipError_t launch_empty_probe(void *, int, hipStream_t) { return hipSuccess; }
}
"""


@functools.lru_cache(1)
def _library():
    """Built once per state of its sources and kept beside the tests, so that a machine that is handed the tree need not
    compile anything."""
    text = LAUNCHERS + "".join(open(os.path.join(build.CSRC, f)).read() for f in ["relay_attn.hip"] + build.HEADERS)
    name = hashlib.sha256((text + " ".join(build.FLAGS)).encode()).hexdigest()[:16]
    out = os.path.join(os.path.dirname(os.path.abspath(__file__)), "_build", "launches_%s.so" % name)
    if not os.path.exists(out):
        os.makedirs(os.path.dirname(out), exist_ok=True)
        with tempfile.TemporaryDirectory(dir=os.path.dirname(out)) as tmp:
            src, new = os.path.join(tmp, "launchers.hip"), os.path.join(tmp, "recorded.so")
            with open(src, "w") as f:
                f.write(LAUNCHERS)
            r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS +
                               ["-Wl,-Bsymbolic", "-I", build.CSRC, os.path.join(build.CSRC, "relay_attn.hip"), src, "-o", new],
                               capture_output=True, text=True)
            assert r.returncode == 0, r.stderr[-2000:]
            for old in os.listdir(os.path.dirname(out)):
                if old.startswith("launches_"):
                    os.unlink(os.path.join(os.path.dirname(out), old))
            os.replace(new, out)
    lib = ctypes.CDLL(out)
    lib.take_launches.restype = ctypes.c_char_p
    lib.relay_attn_workspace_bytes.restype = ctypes.c_size_t
    return lib


AT = ctypes.c_void_p(1 << 20)          # stands for every device address: nothing follows it
SIZE = ctypes.c_size_t


def _launches(lib, status):
    taken = json.loads(lib.take_launches())
    assert status == ra.binding.RA_OK, status
    return taken


def workspace_bytes(p, total_q=None):
    return int(_library().relay_attn_workspace_bytes(ctypes.byref(p), p.batch if total_q is None else total_q))


def decode(p, workspace=None):
    lib = _library()
    size = SIZE(workspace_bytes(p) if workspace is None else workspace)
    return _launches(lib, lib.relay_attn_decode(ctypes.byref(p), *[AT] * 10, size, None))


def _prefixes(lens, counts):
    arr, at = (binding.RAPrefix * len(lens))(), 0
    for f, n, count in zip(arr, lens, counts):
        f.k_sys = f.v_sys = AT if n else None
        f.sys_len, f.first_request, f.num_requests = n, at, count
        at += count
    return arr


def decode_multi(p, lens, counts, workspace=None):
    lib = _library()
    size = SIZE(workspace_bytes(p) if workspace is None else workspace)
    return _launches(lib, lib.relay_attn_decode_multi(ctypes.byref(p), len(lens), _prefixes(lens, counts), *[AT] * 8, size, None))


def decode_grouped(p, lens, counts, workspace=None):
    lib = _library()
    size = SIZE(workspace_bytes(p) if workspace is None else workspace)
    return _launches(lib, lib.relay_attn_decode_grouped(ctypes.byref(p), len(lens), _prefixes(lens, counts), *[AT] * 10, size, None))


def prefill(p, total_q, max_q, workspace=None):
    lib = _library()
    size = SIZE(workspace_bytes(p, total_q) if workspace is None else workspace)
    return _launches(lib, lib.relay_attn_prefill(ctypes.byref(p), AT, AT, total_q, max_q, *[AT] * 9, size, None))


def prefill_multi(p, lens, counts, tokens, max_q, workspace=None):
    lib, total_q = _library(), sum(tokens)
    size = SIZE(workspace_bytes(p, total_q) if workspace is None else workspace)
    toks = (ctypes.c_int32 * len(tokens))(*tokens)
    return _launches(lib, lib.relay_attn_prefill_multi(ctypes.byref(p), len(lens), _prefixes(lens, counts), toks, AT, AT,
                                                       total_q, max_q, *[AT] * 7, size, None))


LATE_BYTES = 12 << 20


def late_payloads(fuse, head_dim):
    """Whether the fusion loads payloads behind the likely ones after their log-sum-exps (the rule in fuse.hip)."""
    first = 8 * (1024 // head_dim if fuse["partials"] > 16 and fuse["rows"] <= 2048 else 1)
    return (min(fuse["partials"], first) - fuse["likely"]) * fuse["rows"] * head_dim * 4 > LATE_BYTES
