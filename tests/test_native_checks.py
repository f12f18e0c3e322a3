"""Host-only native checks (no GPU): the oracle's C code under AddressSanitizer and
UndefinedBehaviorSanitizer, and the unit test of the launch-limit rule the library applies before
it accepts a state."""
import itertools
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")


def _run(cmd, env=None, timeout=600):
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=timeout, env=env)
    assert res.returncode == 0, f"{' '.join(cmd)}\n{res.stdout[-3000:]}\n{res.stderr[-3000:]}"
    return res.stdout + res.stderr


def test_oracle_is_clean_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    exe = str(tmp_path / "oracle_sanitizer_run")
    srcs = [os.path.join(ROOT, "oracle", f) for f in ("philox.c", "classic.c", "craftax_full.c")]
    _run(["gcc", "-O1", "-g", "-std=c11", "-ffp-contract=off", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
          "-static-libasan", "-o", exe, os.path.join(NATIVE, "oracle_sanitizer_run.c")] + srcs + ["-lm"])
    env = dict(os.environ)                          # the sanitizer runtime is linked statically: whatever is preloaded stays
    env["ASAN_OPTIONS"] = "detect_leaks=0:abort_on_error=0"
    env["UBSAN_OPTIONS"] = "print_stacktrace=1"
    out = _run([exe], env=env)
    assert "oracle_sanitizer_run: ok" in out and "runtime error" not in out and "AddressSanitizer" not in out, out[-3000:]


def test_regeneration_units_are_dealt_out_exactly_once(tmp_path):
    """The walk that shares the regeneration units of a step launch between its blocks (csrc/regen_units.hpp)."""
    exe = str(tmp_path / "regen_units_test")
    _run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-o", exe, os.path.join(NATIVE, "regen_units_test.cpp")])
    assert "regen_units_test: ok" in _run([exe])


def test_every_wavefront_of_a_launch_sees_its_number(tmp_path):
    """The launch bookkeeping (csrc/lookahead.hpp) with any one wavefront served last, on the host."""
    exe = str(tmp_path / "launch_order_test")
    _run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-Wno-unknown-pragmas", "-I", os.path.join(NATIVE, "host_hip"), "-o", exe,
          os.path.join(NATIVE, "launch_order_test.cpp")])
    assert "launch_order_test: ok" in _run([exe])


def test_carry_masks_of_the_generators_come_from_a_scalar_instruction(tmp_path):
    """The generators' inline assembly, as compiled: an addition whose carry is a mask in scalar registers has
    it from a scalar instruction of the same statement.  What a vector instruction has just written there is not ready for the
    next two, and the compiler does not look into the statement."""
    src = tmp_path / "generators.hip"
    csrc = os.path.join(ROOT, "paper_2402_16801_amd", "csrc")
    src.write_text('''#include "worldgen.hpp"
#include "full_common.hpp"
#include "full_worldgen.hpp"
template <bool PERLIN> __global__ void classic(uint8_t* maps, const uint32_t* cs)
{
    __shared__ uint32_t lat[cx::LAT_WORDS];
    cx::worldgen_block<512, PERLIN>(maps, lat, 1u, 2u, 3u, 4u, nullptr, 0, cs);
}
template <bool PERLIN> __global__ void floors(uint8_t* maps, const uint32_t* cs)
{
    __shared__ uint32_t lat[cf::LAT_WORDS];
    __shared__ cf::GenLayout layout;
    cf::worldgen_floor_block<64, PERLIN>(maps, lat, layout, 1u, 2u, 3u, 4u, (int)blockIdx.x, nullptr, nullptr, cs);
}
template __global__ void classic<false>(uint8_t*, const uint32_t*);
template __global__ void classic<true>(uint8_t*, const uint32_t*);
template __global__ void floors<false>(uint8_t*, const uint32_t*);
template __global__ void floors<true>(uint8_t*, const uint32_t*);
''')
    out = tmp_path / "generators.s"
    from paper_2402_16801_amd.build import HIPCC_FLAGS

    _run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")] +
         ["-I", csrc, "-S", "--cuda-device-only", "-o", str(out), str(src)])
    statements = re.findall(r";#?\s*APP\n(.*?);#?\s*NO_APP", out.read_text().replace("#ASMSTART", " APP").replace("#ASMEND", " NO_APP"), re.S)
    adds = 0
    for statement in statements:
        lines = [line.split(";")[0].strip() for line in statement.splitlines() if line.split(";")[0].strip()]
        for i, line in enumerate(lines):
            m = re.match(r"v_addc_co_u32_e64 \S+ \S+ \S+ \S+ (s\[\d+:\d+\]|vcc)$", line.replace(",", " ").replace("  ", " "))
            if not line.startswith("v_addc_co_u32_e64"):
                continue
            adds += 1
            assert m and i > 0 and re.match(r"s_\w+_b64 " + re.escape(m.group(1)) + ",", lines[i - 1]), statement
    assert adds > 8 * 2 * (5 + 3 + 3 + 3), adds


def test_fields_are_computed_between_the_changes_of_the_rounding(tmp_path):
    """The generators as compiled: nothing but conversions of whole numbers in 32-bit floating point in front of the change to
    "towards minus infinity", and nothing at all behind the change back.  The source ties both ends to values and stores; what
    the compiler makes of it is seen here."""
    src = tmp_path / "fields.hip"
    csrc = os.path.join(ROOT, "paper_2402_16801_amd", "csrc")
    arguments = "(uint8_t*, uint32_t, uint32_t, const uint32_t*)"
    instances = [f"classic<{nt}, {p}, {s}>" for nt, s in ((256, "false"), (256, "true"), (512, "true")) for p in ("false", "true")]
    instances += [f"floors<{nt}, {p}>" for nt in (64, 320) for p in ("false", "true")]
    src.write_text('''#include "worldgen.hpp"
#include "full_common.hpp"
#include "full_worldgen.hpp"
template <int NT, bool PERLIN, bool SPLIT> __global__ void classic(uint8_t* maps, uint32_t lo, uint32_t hi, const uint32_t* cs)
{
    __shared__ uint32_t lat[cx::LAT_WORDS];
    cx::worldgen_block<NT, PERLIN, SPLIT>(maps, lat, lo, hi, blockIdx.x, 4u, nullptr, 0, cs);
}
template <int NT, bool PERLIN> __global__ void floors(uint8_t* maps, uint32_t lo, uint32_t hi, const uint32_t* cs)
{
    __shared__ uint32_t lat[cf::LAT_WORDS];
    __shared__ cf::GenLayout layout;
    cf::worldgen_floor_block<NT, PERLIN>(maps, lat, layout, lo, hi, blockIdx.x, 4u, (int)blockIdx.y, nullptr, nullptr, cs);
}
''' + "".join(f"template __global__ void {i}{arguments};\n" for i in instances))
    out = tmp_path / "fields.s"
    from paper_2402_16801_amd.build import HIPCC_FLAGS

    _run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")] +
         ["-I", csrc, "-S", "--cuda-device-only", "-o", str(out), str(src)])
    kernels = re.findall(r"^(_Z\S+):(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)
    assert len(kernels) == len(instances)
    for name, body in kernels:
        lines = [line.split(";")[0].strip() for line in body.splitlines()]
        modes = [i for i, line in enumerate(lines) if line.startswith("s_setreg")]
        assert len(modes) == 2 and lines[modes[0]].endswith(", 2") and lines[modes[1]].endswith(", 0"), (name, [lines[i] for i in modes])
        floats = [i for i, line in enumerate(lines) if re.match(r"v_\w*f32", line)]
        assert sum(modes[0] < i < modes[1] for i in floats) > 200, name
        assert [lines[i] for i in floats if i < modes[0] and not lines[i].startswith("v_cvt_f32_")] == [], name
        assert [lines[i] for i in floats if i > modes[1]] == [], name


def test_floors_go_to_the_form_that_was_measured_faster(tmp_path):
    """Blocks or single wavefronts for the floors of a call (csrc/floor_route.hpp)."""
    exe = str(tmp_path / "floor_route_test")
    _run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-o", exe, os.path.join(NATIVE, "floor_route_test.cpp")])
    assert "floor_route_test: ok" in _run([exe])


def test_worlds_owed_by_a_rollout_go_where_it_was_measured_faster(tmp_path):
    """A launch behind a Classic rollout or its own blocks (csrc/rollout_route.hpp)."""
    exe = str(tmp_path / "rollout_route_test")
    _run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-o", exe, os.path.join(NATIVE, "rollout_route_test.cpp")])
    assert "rollout_route_test: ok" in _run([exe])


def test_public_header_compiles_as_c_and_as_cpp(tmp_path):
    """include/craftax.h on its own, with warnings as errors, as C11 and as C++17: no HIP or torch type
    in any signature, every struct complete."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    body = '#include "craftax.h"\nint main(void) { craftax_config c; craftax_metrics m; (void)c; (void)m; return (int)sizeof(craftax_metrics) == 0; }\n'
    for name, cc, std in (("use.c", "gcc", "-std=c11"), ("use.cpp", "g++", "-std=c++17")):
        src = tmp_path / name
        src.write_text(body)
        _run([cc, std, "-Wall", "-Wextra", "-Werror", "-pedantic", "-I", os.path.join(root, "include"), "-c", "-o", str(tmp_path / (name + ".o")), str(src)])


def test_launch_limit_rule(tmp_path):
    exe = str(tmp_path / "launch_limits_test")
    _run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-o", exe, os.path.join(NATIVE, "launch_limits_test.cpp")])
    assert "launch_limits_test: ok" in _run([exe])


def _kernel_instances(text):
    """`kf_name<arguments>` in a piece of the host code, template parameters of the enclosing function as both of their values."""
    out = set()
    for name, args in re.findall(r"\b(kf_\w+)\s*(<[^<>;]*>)?", text):
        args = [a.strip() for a in args.strip("<>").split(",")] if args else []
        for values in itertools.product(*[("true", "false") if a in ("F32", "PERLIN") else (a,) for a in args]):
            out.add((name,) + values)
    return out


def test_every_kernel_the_full_game_launches_is_checked_against_the_device():
    """The full game's host code in csrc/full.hip: every kernel instance it launches is one that a state
    is refused for if the device cannot launch it."""
    src = open(os.path.join(ROOT, "paper_2402_16801_amd", "csrc", "full.hip")).read()
    host = re.sub(r"//[^\n]*", "", src[src.index("namespace host {"):])
    host = re.sub(r'"[^"\n]*"', "", host)
    check = re.search(r"static bool kernels_fit\b.*?\n}\n", host, re.S).group(0)
    asked, launched = _kernel_instances(check), _kernel_instances(host.replace(check, ""))
    assert len(launched) > 20 and launched <= asked, sorted(launched - asked)


def test_noise_fields_equal_the_oracle(tmp_path):
    """The generators' fields in floating point rounded down (csrc/noise_fields.hpp) against the oracle's integers."""
    exe, objs = str(tmp_path / "noise_fields_test"), []
    for name in ("philox", "classic"):
        objs.append(str(tmp_path / f"{name}.o"))
        _run(["gcc", "-O2", "-std=c11", "-ffp-contract=off", "-c", "-o", objs[-1], os.path.join(ROOT, "oracle", name + ".c")])
    _run(["g++", "-O2", "-march=native", "-frounding-math", "-ffp-contract=off", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-o", exe,
          os.path.join(NATIVE, "noise_fields_test.cpp")] + objs + ["-lm"])
    assert "noise_fields_test: ok" in _run([exe])
