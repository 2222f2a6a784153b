#!/bin/bash
# Builds libkdloss.so for gfx950 next to the sources, the source files side by side.
set -e
cd "$(dirname "$0")"
FLAGS="--offload-arch=gfx950 -O3 -std=c++17 -fPIC -Xclang -target-feature -Xclang -packed-fp32-ops"
OBJ=$(mktemp -d)
trap 'rm -rf "$OBJ"' EXIT
pids=()
for f in kd_kernels kd_strip_hv kd_products kd_few kd_api; do
  hipcc $FLAGS "$@" -c $f.hip -o "$OBJ/$f.o" & pids+=($!)
done
for p in "${pids[@]}"; do wait $p; done
hipcc --offload-arch=gfx950 -shared "$OBJ"/*.o -o libkdloss.so
