"""Nothing that belongs to a device is kept per process: which kernels may take how much LDS is asked for once per device,
under a lock, by the first ccld_create on it (a source check: it runs without a GPU)."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_04478_amd", "csrc")
FILES = {n: re.sub(r"//.*", "", open(os.path.join(CSRC, n)).read()) for n in sorted(os.listdir(CSRC)) if n.endswith((".hip", ".h"))}


@pytest.mark.parametrize("name", sorted(FILES))
def test_no_mutable_statics_in_functions(name):
    assert re.findall(r"^[ \t]+static (?!constexpr|const |inline|__device__)[^;()]*;", FILES[name], flags=re.M) == []


def test_create_asks_for_every_kernel_with_more_lds_than_the_default():
    assert "ccld_device_init()" in FILES["api.hip"].split("ccld_status ccld_create(")[1].split("ccld_status ccld_destroy(")[0]
    assert "device_scratch(" in FILES["hang.hip"].split("ccld_status ccld_device_init() {")[1].split("}")[0]
    first = FILES["hang.hip"].split("ccld_status device_scratch(")[1].split("\n}")[0]
    assert first.index("lock_guard") < first.index("allow_lds") < first.index("g_scratch_ptr[dev] =")
    for name, text in FILES.items():
        fn = re.findall(r"hipError_t (?:ccld::)?(allow_lds_\w+)\(\) \{", text)
        assert len(fn) == len(re.findall(r"hipError_t (?:ccld::)?allow_lds_\w+\(\) \{", text)) <= 1
        for f in fn:
            assert f + "()" in first, (name, f)
        # nobody else sets the attribute
        assert text.count("hipFuncSetAttribute") == (1 if name == "ccld_internal.h" else 0), name
