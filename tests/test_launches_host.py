"""The host half of the calls without a GPU: the library in a process whose HIP
runtime is a stand-in that records launches and allocations and runs nothing,
so that what a call enqueues can be compared with what the device will need."""
import json
import os
import subprocess
import sys

import pytest

from paper_2608_09225_amd import kvgov as K

pytestmark = pytest.mark.skipif(not os.path.exists(K.LIB_PATH), reason="libkvgov.so not built")

RUNTIME = r"""
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
static std::map<const void *, std::string> names;
static std::string launched;
static int capturing = 0;
static size_t fail_bytes = 0;
// the epochs that kernels are launched with
static std::string epochs;
static void note_epoch(const std::string &k, void **args) {
  const char *by[] = {"k_insert_req", "k_chunk_insert", "k_reinsert", "k_radix_roots"};
  const int at[] = {5, 5, 5, 3};
  for (int i = 0; i < 4; ++i)
    if (k.find(by[i]) != std::string::npos)
      epochs += std::to_string(*(const uint32_t *)args[at[i]]) + " ";
}
extern "C" {
void *__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterFunction(void *, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) { names[host] = name; }
void __hipRegisterVar(void *, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void *) {}
struct Dim { uint32_t x, y, z; };
static Dim grid_, block_; static size_t shmem_; static void *stream_;
int __hipPushCallConfiguration(Dim g, Dim b, size_t s, void *st) {
  grid_ = g; block_ = b; shmem_ = s; stream_ = st; return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *s, void **st) {
  *g = grid_; *b = block_; *s = shmem_; *st = stream_; return 0; }
// of a clear, also whether it writes the recency words (the second array of its zeros)
int hipLaunchKernel(const void *f, Dim, Dim, void **args, size_t, void *) {
  launched += names[f] + "\n";
  if (names[f].find("k_cache_fill") != std::string::npos && ((int64_t *)args[0])[8])
    launched += "k_recencyE\n";
  note_epoch(names[f], args);
  return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipFree(void *p) { free(p); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **, const void *) { return 1; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return 0; }
int hipMalloc(void **p, size_t n) {
  if (fail_bytes && n >= fail_bytes) return 2;
  *p = malloc(64); return 0; }
int hipMemcpyAsync(void *d, const void *, size_t n, int, void *) { memset(d, 0, n); return 0; }
int hipMemset(void *, int, size_t) { return 0; }
int hipStreamIsCapturing(void *, int *s) { *s = capturing; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipThreadExchangeStreamCaptureMode(int *) { return 0; }
void test_capture(int on) { capturing = on; }
const char *test_epochs() { static std::string s; s = epochs; epochs.clear(); return s.c_str(); }
void test_fail_from(size_t bytes) { fail_bytes = bytes; }
const char *test_launched() { static std::string s; s = launched; launched.clear(); return s.c_str(); }
}
"""

PRELUDE = """
import ctypes, json, re
hip = ctypes.CDLL({hip!r}, mode=ctypes.RTLD_GLOBAL)
hip.test_launched.restype = ctypes.c_char_p
hip.test_epochs.restype = ctypes.c_char_p
lib = ctypes.CDLL({lib!r})
i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
fake = vp(0x1000)  # device memory: never touched here
def launched():
    return re.findall(r"(k_\\w+?)(?:I[LN]|E)", hip.test_launched().decode())
def epochs():
    return [int(e) for e in hip.test_epochs().split()]
def cache(log2_slots, track=1):
    h = vp()
    assert lib.kvgov_cache_create(i32(log2_slots), ctypes.byref(h)) == 0
    assert lib.kvgov_cache_set_recency(h, i32(track)) == 0
    return h
def insert(h, n, n_blocks):
    assert lib.kvgov_cache_insert(h, fake, fake, i32(n), i64(n_blocks), None, None) == 0
def clear(h):
    assert lib.kvgov_cache_clear(h, None) == 0
def evict(h):
    launched()
    assert lib.kvgov_cache_evict(h, i64(10), None, None) == 0
    return launched()
launched()
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("launches")
    src, out = d / "hip.cpp", d / "libhip_stand_in.so"
    src.write_text(RUNTIME)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(out), str(src)], check=True)

    def go(body):
        script = PRELUDE.format(hip=str(out), lib=K.LIB_PATH) + body
        r = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.splitlines()[-1])

    return go


def passes(bits):
    return max(1, -(-bits // 11))  # bits that one pass of the select decides


def test_evict_decides_every_bit_that_can_differ(run):
    """An eviction's passes cover the stamps and depths that any call so far has
    been given, captured ones that run after a clear included; a captured
    eviction covers whole words."""
    got = run("""
out = {}
h = cache(16)
out["empty"] = evict(h).count("k_rank_select")
for _ in range(4000):
    insert(h, 3, 20)
insert(h, 3, 5000)
out["filled"] = evict(h).count("k_rank_select")
clear(h)
out["unused"] = evict(h).count("k_rank_select")
for _ in range(4000):
    insert(h, 3, 20)
hip.test_capture(1)
insert(h, 3, 5000)
hip.test_capture(0)
clear(h)  # the graph may insert with the stamp of its capture
out["cleared"] = evict(h).count("k_rank_select")
hip.test_capture(1)
out["captured"] = evict(h).count("k_rank_select")
print(json.dumps(out))
""")
    need = passes((4001).bit_length() + (5000).bit_length())
    assert got["empty"] == got["unused"] == 1
    assert got["filled"] == need
    assert got["cleared"] >= need
    assert got["captured"] == passes(64)


def test_captured_clear_leaves_the_host_state(run):
    """A clear that is being captured has emptied nothing: the next insert takes a
    new epoch, and every run of the graph writes the recency words, whatever the
    table held at the capture."""
    got = run("""
out = {}
h = cache(16)
clear(h); launched()
clear(h); out["unused"] = launched()
for _ in range(1000):
    insert(h, 3, 20)
out["passes"] = evict(h).count("k_rank_select")
clear(h); out["used"] = launched()
hip.test_capture(1)
clear(h); out["captured"] = launched()
insert(h, 3, 20); launched()
hip.test_capture(0)
clear(h); out["after"] = launched()
print(json.dumps(out))
""")
    assert got["unused"] == ["k_cache_fill"]
    assert got["used"] == got["captured"] == got["after"] == ["k_cache_fill", "k_recency"]


@pytest.mark.parametrize("call", ["insert", "admit", "evict", "radix"])
def test_clears_of_a_table_that_a_graph_stamps(run, call):
    """Once a call that stamps keys has been captured its graph may run between
    any two calls: every clear writes the recency words and sets the clock back, and
    no later call of the table gets the graph's epoch."""
    got = run("""
def radix_insert(x):
    assert lib.kvgov_radix_insert(x, fake, i64(40), fake, i32(2), None, None, i32(0), i32(0),
                                  fake, fake, i64(2), None) == 0
def admit(h):
    assert lib.kvgov_cache_admit(h, fake, fake, i32(3), i64(20), fake, fake, None, None) == 0
call = {call!r}
if call == "radix":
    h = vp()
    assert lib.kvgov_radix_create(i32(10), i32(10), ctypes.byref(h)) == 0
    stamp, wipe = radix_insert, lambda h: lib.kvgov_radix_clear(h, None)
else:
    h, wipe = cache(16), lambda h: lib.kvgov_cache_clear(h, None)
    stamp = {{"insert": lambda h: insert(h, 3, 20), "admit": admit, "evict": evict}}[call]
stamp(h); wipe(h); launched(); hip.test_epochs()
wipe(h)
out = {{"before": launched()}}
stamp(h); out["first"] = epochs()
wipe(h); stamp(h); out["again"] = epochs()
hip.test_capture(1)
stamp(h); out["graph"] = epochs()
hip.test_capture(0)
out["clears"] = []
for _ in range(3):
    wipe(h); launched()
    wipe(h); out["clears"].append(launched())
    for _ in range(5):
        stamp(h)
out["later"] = epochs()
print(json.dumps(out))
""".format(call=call))
    assert got["before"] == ["k_cache_fill"]
    assert got["first"] == got["again"]  # a clear starts the clock again
    assert got["clears"] == [["k_cache_fill", "k_recency"]] * 3
    assert not set(got["graph"]) & set(got["later"])
    assert len(set(got["later"])) == len(got["later"]) // 3  # and each clear starts it again


def test_radix_create_without_memory_for_chains(run):
    """An index whose tables can be had is created, with or without the records
    of chains; one whose tables cannot be had is refused."""
    got = run("""
def create(fail_from):
    hip.test_fail_from(ctypes.c_size_t(fail_from))
    x = vp()
    rc = lib.kvgov_radix_create(i32(20), i32(18), ctypes.byref(x))
    hip.test_fail_from(ctypes.c_size_t(0))
    if rc == 0:
        assert lib.kvgov_radix_insert(x, fake, i64(40), fake, i32(2), None, None, i32(0), i32(0),
                                      fake, fake, i64(2), None) == 0
        assert lib.kvgov_radix_clear(x, None) == 0
        assert lib.kvgov_radix_destroy(x) == 0
    return rc
print(json.dumps([create(n) for n in (0, 64 << 20, 8 << 20, 2 << 20)]))
""")
    c = K.header_constants()
    assert got == [0, 0, c["KVGOV_E_NOMEM"], c["KVGOV_E_NOMEM"]]
