"""What a sky's calls write while another thread may read it: the kernel duration
that fgl_sky_kernel_ms returns without the sky's lock is an atomic.  Read from the
source: a torn or stale value can't be provoked."""
import re

from tests.test_wave_exchange_cpu import _body, _code


def test_kernel_ms_is_read_without_a_race():
    code = _code("fgl_sky.hip")
    assert re.search(r"std::atomic<double>\s+last_ms", code)
    assert "last_ms" in _body(code, "int fgl_sky_kernel_ms(")
