"""Every variant of the stage kernel in the gfx950 assembly of the library build
(CPU only: cross-compiles, needs hipcc): the one-plane kernels take one struct
at offset 0 and use the scalar-base form in their march, as test_kernel_args.py
says of the general ones, and no variant spills more vector registers than the
comment at stage_threads states."""
import re

from test_kernel_args import kernel_args, plane_loop, segment_loads

# vector registers spilled: [general, one plane] of the variants
# <real, gas + radiation, optional features>
SPILLED = {"dLb0ELb0": (0, 0), "dLb0ELb1": (16, 27), "dLb1ELb0": (7, 50), "dLb1ELb1": (34, 50),
           "fLb0ELb0": (0, 0), "fLb0ELb1": (3, 9), "fLb1ELb0": (3, 0), "fLb1ELb1": (13, 26)}


def test_plane_kernels_take_one_struct_at_offset_zero(kernels_asm):
    kern = kernel_args(kernels_asm, r"^_ZN3mhd18plane_stage_kernelI")
    assert len(kern) == 8, sorted(kern)
    for name, args in kern.items():
        explicit = [a for a in args if not a[2].startswith("hidden_")]
        assert len(explicit) == 1, (name, args)
        off, size, kind = explicit[0]
        assert (off, kind) == (0, "by_value"), (name, explicit)
        loads = segment_loads(kernels_asm, name)
        for o, w in loads:
            assert any(a <= o and o + w <= a + n for a, n, _ in args), (name, o, w, args)
        assert any(o + w <= size for o, w in loads), name


def test_plane_kernels_address_from_scalar_bases(kernels_asm):
    for name in kernel_args(kernels_asm, r"^_ZN3mhd18plane_stage_kernelI"):
        loop = plane_loop(kernels_asm, name)
        mem = [x.split(None, 1) for x in loop if re.match(r"\s+global_(load|store)", x)]
        assert len(mem) >= 40, (name, len(mem))
        vec = [m for m in mem if m[1].split(",")[-1].strip().startswith("off")]
        assert not vec, (name, vec[:3])
        if "kernelIf" in name:
            reloads = sum(1 for x in loop if "v_readlane_b32" in x)
            assert reloads <= 4, (name, reloads)


def test_spilled_registers_of_every_variant(kernels_asm):
    seen, cur = {}, {}
    for x in kernels_asm:
        m = re.match(r"\s+(?:- )?\.(name|vgpr_count|vgpr_spill_count):\s+(\S+)$", x)
        if m:
            cur[m.group(1)] = m.group(2)
            if m.group(1) == "vgpr_spill_count":
                k = re.match(r"_ZN3mhd\d+(plane_)?stage_kernelI(\w+)EEEvNS_9StageArgsE$", cur["name"])
                if k:
                    seen[k.group(2), bool(k.group(1))] = (int(cur["vgpr_count"]),
                                                          int(cur["vgpr_spill_count"]))
                cur = {}
    assert len(seen) == 16, sorted(seen)
    for (variant, flat), (count, spilled) in seen.items():
        # three waves per SIMD in FP64, four in FP32
        assert count <= (168 if variant[0] == "d" else 128), (variant, flat, count)
        assert spilled <= SPILLED[variant][flat], (variant, flat, spilled)
