"""The rules of csrc/columns_rule.h (which forward kernels take their tokens in columns), compiled with the host compiler."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include "columns_rule.h"
extern "C" {
int small_columns(int gw, int out_token_stride) { return aa::small_columns(gw, out_token_stride); }
int small_column_segment(int units, int gh, int gw) { return aa::small_column_segment(units, gh, gw, 256); }
int large_column_parts(int n, int gh, int cells) { return aa::large_column_parts(n, gh, cells); }
int large_aggregate_columns(int width, int n, int gh, int gw, int cells) { return aa::large_aggregate_columns(width, n, gh, gw, cells); }
int large_columns_pay(int width, int parts, int n, int units, int gh, int gw) { return aa::large_columns_pay(width, parts, n, units, gh, gw, 256); }
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
