"""The rules of csrc/columns_rule.h (which forward kernels take their tokens in columns) and csrc/split_rules.h (blocks of the
projections and of the one-launch fp32 kernel), compiled with the host compiler."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include "columns_rule.h"
#include "split_rules.h"
extern "C" {
int small_columns(int gw, int out_token_stride) { return aa::small_columns(gw, out_token_stride); }
int small_column_segment(int units, int gh, int gw) { return aa::small_column_segment(units, gh, gw, 256); }
int large_column_parts(int n, int gh, int cells) { return aa::large_column_parts(n, gh, cells); }
int large_aggregate_columns(int width, int n, int gh, int gw, int cells) { return aa::large_aggregate_columns(width, n, gh, gw, cells); }
int large_columns_pay(int width, int parts, int n, int units, int gh, int gw) { return aa::large_columns_pay(width, parts, n, units, gh, gw, 256); }
void projection_blocks(long long M, int O, int K, int* out) {
  const aa::ProjectionBlocks b = aa::projection_blocks(M, O, K, 256);
  out[0] = b.rows, out[1] = b.outputs, out[2] = b.step;
}
void fused_f32_shares(int N, int d, int units, int* out) {
  const aa::UnitShares s = aa::fused_f32_shares(N, d, units, 256);
  out[0] = s.tiles, out[1] = s.parts, out[2] = s.channel_tiles;
}
}
'''


def load(folder):
    src, lib = os.path.join(folder, "columns_rule.cpp"), os.path.join(folder, "columns_rule.so")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2312_08874_amd", "csrc"),
                    "-o", lib, src], check=True)
    return ctypes.CDLL(lib)


def large_parts(rules, grid, n, d, units, cells):
    """Cell rows in a stage of the column kernel that serves a problem, 0: the rows kernel does."""
    parts = rules.large_column_parts(n, grid[0], cells) if grid[1] % 4 == 0 else 0
    width = 32 if d <= 32 else 64 if d <= 64 else 128
    return parts if parts and rules.large_columns_pay(width, parts, n, units, *grid) else 0


def aggregate_columns(rules, grid, n, d, cells):
    """Whether the aggregation of a problem with half-resized tables takes its tokens in columns."""
    return grid[1] % 4 == 0 and n > 64 and bool(rules.large_aggregate_columns(32 if d <= 32 else 64 if d <= 64 else 128, n, *grid, cells))


def projection_blocks(rules, rows, outputs, channels):
    """(rows, outputs) of a block and channels of a step of a product."""
    out = (ctypes.c_int * 3)()
    rules.projection_blocks(ctypes.c_longlong(rows), outputs, channels, out)
    return tuple(out)


def fused_f32_shares(rules, N, d, units):
    """(blocks along a unit's tokens, 16-channel tiles a block takes)."""
    out = (ctypes.c_int * 3)()
    rules.fused_f32_shares(N, d, units, out)
    return tuple(out)[1:]
