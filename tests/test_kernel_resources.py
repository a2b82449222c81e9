"""What the host and the device code assume about the compiled kernels, read from the metadata of the code objects in the
built library (registers and LDS per workgroup; no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2604_07394_amd", "lib", "libflux.so")
READELF = "/opt/rocm/lib/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: metadata} of every gfx950 kernel of the library."""
    if not os.path.exists(LIB):
        from paper_2604_07394_amd import build
        build.build_all()
    blob = open(LIB, "rb").read()
    found = {}
    at = blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", blob, at + len(MAGIC))[0]):
            offset, size, n = struct.unpack_from("<QQQ", blob, pos)
            triple = blob[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" not in triple or size == 0:
                continue
            obj = tmp_path_factory.mktemp("obj") / "code.o"
            obj.write_bytes(blob[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n  - \.", notes)[1:]:
                get = lambda key: re.search(r"\.?" + key + r":\s*(\S+)", part)
                if get("name") and get("vgpr_count"):
                    found[get("symbol").group(1)] = {k: int(get(k).group(1)) for k in ("vgpr_count", "max_flat_workgroup_size", "group_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count")}
        at = blob.find(MAGIC, at + 1)
    return found


def workgroups_per_cu(k):
    """512 registers per SIMD lane, handed out to a wave in steps of 8; four SIMDs and 160 KB of LDS per CU."""
    waves = 4 * (512 // (-(-k["vgpr_count"] // 8) * 8))
    return min(waves // (k["max_flat_workgroup_size"] // 64), 163840 // max(1, k["group_segment_fixed_size"]))


def test_every_decode_kernel_holds_the_round_its_calls_are_made_for(kernels):
    """A decode call launches up to 512 workgroups (2^kDecodeAlignedShift of four waves, kDecodeFewWgs of eight) that are meant
    to run side by side, two per CU on 256 CUs: no instance may need more registers or LDS than that leaves, or spill."""
    src = open(os.path.join(ROOT, "paper_2604_07394_amd", "csrc", "flux_internal.h")).read()
    most = {256: 1 << int(re.search(r"kDecodeAlignedShift = (\d+);", src).group(1)), 512: int(re.search(r"kDecodeFewWgs = (\d+);", src).group(1))}
    names = [n for n in kernels if "decode_splitk_kernel" in n]
    assert sorted(kernels[n]["max_flat_workgroup_size"] for n in names) == [256] * 12 + [512] * 6
    for n in names:
        assert 256 * workgroups_per_cu(kernels[n]) >= most[kernels[n]["max_flat_workgroup_size"]] >= 512, (n, kernels[n])
        assert kernels[n]["vgpr_spill_count"] == 0, n


def test_every_prefill_kernel_holds_the_workgroups_its_launches_count_on(kernels):
    """The rules of a prefill launch (which tiles, whether keys are shared out) count on kResident128 workgroups side by side at
    head dimension 128 and kResident64 at 64.  prefill.hip is compiled with regions left unstructurised, which is what keeps the
    registers of its loops down: no instance may spill."""
    src = open(os.path.join(ROOT, "paper_2604_07394_amd", "csrc", "prefill.hip")).read()
    names = [n for n in kernels if "prefill_kernel" in n]
    assert len(names) == 10
    for n in names:
        d = 128 if "ILi128E" in n else 64
        resident = int(re.search(r"kResident%d = (\d+)" % d, src).group(1))
        assert 256 * workgroups_per_cu(kernels[n]) >= resident >= 512, (n, kernels[n])
        assert kernels[n]["vgpr_spill_count"] == 0 and kernels[n]["sgpr_spill_count"] == 0, (n, kernels[n])


def test_router_launches_of_many_workgroups_run_an_instance_that_shares_the_cus(kernels):
    """An MLP workgroup that keeps rounds of 4096 columns in registers leaves room for two per CU.  The instance for many
    workgroups and for narrow layers holds five."""
    k = [v for n, v in kernels.items() if "router_mlp_kernelILi1024E" in n]
    assert len(k) == 1 and workgroups_per_cu(k[0]) >= 5 and k[0]["vgpr_spill_count"] == 0, k


def test_counter_records_belong_to_the_compiler_flags_too(monkeypatch):
    """bench.py reports recorded counters while the digest of their kernel holds: flags change a kernel as its source does."""
    import bench
    from paper_2604_07394_amd import build
    names = ["prefill.hip", "flux_internal.h"]
    before = bench.source_digest(names)
    assert before == bench.source_digest(names)
    monkeypatch.setattr(build, "SOURCE_FLAGS", {})
    assert bench.source_digest(names) != before
    monkeypatch.undo()
    monkeypatch.setattr(build, "COMMON", build.COMMON + ["-O2"])
    assert bench.source_digest(names) != before
