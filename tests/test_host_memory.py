"""Running out of host memory is an error code at the C boundary, not an exception
that ends the caller's process."""
import subprocess
import sys

CHILD = """
import ctypes, resource
from paper_1106_2899_amd import _lib as L
so = L.lib()
c = L.SspConfig()
so.ssp_config_init(ctypes.byref(c))
c.n_chains = c.n_elements = 1 << 28  # 1 GB for the chains' lengths alone
c.corr_levels = 0
sb, wb = ctypes.c_size_t(), ctypes.c_size_t()
with open("/proc/self/statm") as f:
    now = int(f.read().split()[0]) * resource.getpagesize()
old = resource.getrlimit(resource.RLIMIT_AS)
resource.setrlimit(resource.RLIMIT_AS, (now + (1 << 28), old[1]))
rc = so.ssp_query_sizes(ctypes.byref(c), ctypes.byref(sb), ctypes.byref(wb))
resource.setrlimit(resource.RLIMIT_AS, old)
print(rc, so.ssp_last_error(None).decode())
c.n_chains = c.n_elements = 16
print(so.ssp_query_sizes(ctypes.byref(c), ctypes.byref(sb), ctypes.byref(wb)), sb.value > 0)
"""


def test_out_of_host_memory_is_an_error_code():
    r = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    refused, after = r.stdout.splitlines()
    assert refused == "-1 out of host memory"
    assert after == "0 True"
