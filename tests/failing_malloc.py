"""A hipMalloc that fails when told to, for tests of what the engine does when
device memory runs out.  Loaded ahead of everything that links the runtime, so
use it in a process of its own: ``run(script)`` runs a Python script there, in
which ``failing_malloc.fail(first, count, at_least)`` makes the engine's
first-th to (first + count - 1)-th calls of at least that many bytes report out
of memory, and ``failing_malloc.calls()`` tells how many such calls it made
since.  ``events()`` tells how many events the engine has created, and
``fail_event(n)`` makes its n-th creation from then on (0: the next) fail."""
import ctypes
import os
import subprocess
import sys
import tempfile

TESTS = os.path.dirname(os.path.abspath(__file__))
SOURCE = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <limits.h>
#include <stddef.h>
#include <stdio.h>
#include <string.h>
static size_t least = (size_t)-1;
static long first, count, seen;
void failing_malloc_set(long f, long n, size_t bytes) { first = f; count = n; least = bytes; seen = 0; }
long failing_malloc_calls(void) { return seen; }
static long events, event_in = -1;
long failing_malloc_events(void) { return events; }
void failing_malloc_event(long n) { event_in = n; }
static void *runtime(const char *name) {   /* of the runtime that this process has loaded */
    char line[PATH_MAX + 128], *path;
    void *found = NULL;
    FILE *maps = fopen("/proc/self/maps", "r");
    while (!found && fgets(line, sizeof line, maps)) {
        if (!(path = strchr(line, '/')) || !strstr(path, "libamdhip64")) continue;
        path[strcspn(path, "\n")] = 0;
        void *lib = dlopen(path, RTLD_LAZY | RTLD_NOLOAD);
        if (lib) found = dlsym(lib, name);
    }
    fclose(maps);
    return found;
}
static int engine(void *caller) {
    Dl_info from;
    return dladdr(caller, &from) && strstr(from.dli_fname, "libfl.so");
}
int hipMalloc(void **p, size_t n) {
    static int (*real)(void **, size_t);
    if (!real) *(void **)&real = runtime("hipMalloc");
    if (n >= least && engine(__builtin_return_address(0))) {
        const long at = seen++;
        if (at >= first && at < first + count) { *p = NULL; return 2; }   /* hipErrorOutOfMemory */
    }
    return real(p, n);
}
int hipEventCreate(void **e) {
    static int (*real)(void **);
    if (!real) *(void **)&real = runtime("hipEventCreate");
    if (engine(__builtin_return_address(0))) {
        ++events;
        if (event_in >= 0 && event_in-- == 0) return 2;
    }
    return real(e);
}
"""
_lib = None


def install():
    global _lib
    assert "torch" not in sys.modules and "paper_2210_01465_amd" not in sys.modules
    _lib = ctypes.CDLL(os.environ["FAILING_MALLOC"], mode=ctypes.RTLD_GLOBAL)
    _lib.failing_malloc_set.argtypes = [ctypes.c_long, ctypes.c_long, ctypes.c_size_t]
    _lib.failing_malloc_event.argtypes = [ctypes.c_long]
    _lib.failing_malloc_calls.restype = _lib.failing_malloc_events.restype = ctypes.c_long


def fail(first: int, count: int, at_least: int = 0):
    _lib.failing_malloc_set(first, count, at_least)


def calls() -> int:
    return _lib.failing_malloc_calls()


def events() -> int:
    return _lib.failing_malloc_events()


def fail_event(n: int):
    _lib.failing_malloc_event(n)


def run(script: str, timeout: float = 100):
    """Run the script in a process of its own with the failing hipMalloc; its output."""
    with tempfile.TemporaryDirectory() as tmp:
        src, lib = os.path.join(tmp, "m.c"), os.path.join(tmp, "m.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", src, "-o", lib, "-ldl"], check=True)
        env = dict(os.environ, FAILING_MALLOC=lib, PYTHONPATH=os.pathsep.join([TESTS, os.path.dirname(TESTS)]))
        p = subprocess.run([sys.executable, "-u", "-c", "import failing_malloc\nfailing_malloc.install()\n" + script],
                           env=env, timeout=timeout, capture_output=True, text=True)
    print(p.stdout, p.stderr, flush=True)
    assert p.returncode == 0, p.returncode
    return p.stdout
