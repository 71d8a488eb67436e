// Line lengths the passes are built for.
#pragma once

#define FG_FOR_M(X) X(2) X(3) X(4) X(6) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(256)
// half lines of k_cg_lines
#define FG_FOR_LINES(X) X(2) X(3) X(4) X(6) X(8) X(12) X(16) X(24) X(32)
#define FG_FOR_AXIS(X) X(1) X(4) X(6) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(256)
// N1 passes also take 512-long lines (plane grids of 512 x 512)
#define FG_FOR_N1(X) FG_FOR_AXIS(X) X(512)

