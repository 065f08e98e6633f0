#!/bin/bash
# Builds the host code of the library's sources with AddressSanitizer and UndefinedBehaviorSanitizer (no device code),
# links it with the stand-in for the HIP runtime and the host-only exerciser, and runs that.  No GPU needed.
# $1: where to build (a temporary folder unless given).
set -e
here=$(cd "$(dirname "$0")" && pwd)
root=$(cd "$here/../.." && pwd)
out=${1:-${TMPDIR:-/tmp}/mona_sanitize}
mkdir -p "$out"
src="$root/paper_2605_26842_amd/csrc"
clang=/opt/rocm/lib/llvm/bin/clang++
san="-Xarch_host -fsanitize=address -Xarch_host -fsanitize=undefined -Xarch_host -fno-omit-frame-pointer"
plain="-O1 -g -std=c++17 -fsanitize=address -fsanitize=undefined -fno-omit-frame-pointer -D__HIP_PLATFORM_AMD__ -I/opt/rocm/include"
# every source the library is built from
files=$(cd "$root" && python3 -c 'from paper_2605_26842_amd.build import SOURCES; print(*SOURCES)')
jobs=""; objs=""
for f in $files; do
  o="$out/${f%.hip}.o"
  /opt/rocm/bin/hipcc --offload-arch=gfx950 --offload-host-only -O1 -g -std=c++17 -fPIC -fno-gpu-rdc \
    -Wno-unused-command-line-argument $san -c "$src/$f" -o "$o" > "$o.log" 2>&1 &
  jobs="$jobs $!:$o.log"; objs="$objs $o"
done
# (the stand-in first: the library's objects register their kernels with it before main)
for f in sanitize_host_paths fake_hip; do
  $clang $plain -c "$here/$f.cpp" -o "$out/$f.o" > "$out/$f.o.log" 2>&1 &
  jobs="$jobs $!:$out/$f.o.log"; objs="$out/$f.o $objs"
done
for j in $jobs; do wait "${j%%:*}" || { cat "${j#*:}"; exit 1; }; done
# (there is no device code behind the names under which the objects refer to it)
none=$(nm $objs | awk '$1 == "U" && $2 ~ /^__hip_fatbin/ { print "-Wl,--defsym=" $2 "=0" }')
$clang -fsanitize=address -fsanitize=undefined $objs $none -o "$out/sanitize_host_paths"
ASAN_OPTIONS=detect_leaks=1:abort_on_error=0 UBSAN_OPTIONS=print_stacktrace=1:halt_on_error=1 "$out/sanitize_host_paths"
