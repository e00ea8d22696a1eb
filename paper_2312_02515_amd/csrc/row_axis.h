// Which task a row of a launch belongs to, from the split positions in the kernel arguments (`K`, `off`).
#pragma once

#include "mlora_common.h"

namespace mlora {
namespace rowaxis {

// 32 consecutive rows of the virtual row axis, on which every row range of the call (before the
// first task, each task, after the last) is padded to a multiple of 32: a piece never holds rows of
// two tasks, so no row ever meets another task's adapter, not even multiplied by zero.
struct RowPiece {
  int row, n, task;   // first real row, real rows (0 = beyond the last row), task (-1 = none)
};

// inclusive sums over the first n lanes of a wave
__device__ __forceinline__ int scan_lanes(int v, int n) {
  const int lane = threadIdx.x & 63;
  for (int s = 1; s < n; s <<= 1) {
    const int u = __shfl_up(v, s);
    if (lane >= s) v += u;
  }
  return v;
}

// Up to this many tasks are searched one after the other, by scalar loads; more by all lanes at once: 66
// dependent loads for 64 tasks took 7 us of every block, while the vector loads and the scan cost 1.7 us
// whatever the number of tasks.  Forward and backward in the aligned kernels, one task after the other ->
// by all lanes (ranks up to 64): 2048 rows of 64 tasks, 2048 x 2048  140 -> 112 us, 3000 rows of 40, 3072 x 3072
// 228 -> 217, 1000 rows of 20, 1024 -> 2048  81 -> 77; 300 rows of 10, 4096 x 4096 level.
constexpr int kFewTasks = 8;

// The virtual row axis, spread over a wave: lane k knows where task k stands (all of a wave's lanes call
// this)
struct RowAxis {
  int off, len;                          // task `lane`: first row, rows
  unsigned vlen, vstart;                 // ... rows on the axis, where they start there
  int lead, rows_end, M;                 // rows before the first task, end of the last task's rows
  unsigned vlead, tasks_end;             // ... on the axis
};
template <typename Args>
__device__ __forceinline__ RowAxis row_axis(const Args& a) {
  RowAxis x{};
  if (a.K <= kFewTasks) return x;
  const int lane = threadIdx.x & 63;
  x.off = a.off[lane];                   // (entries from K on repeat the last split position)
  x.len = lane < a.K ? a.off[lane + 1] - x.off : 0;
  x.vlen = ((unsigned)x.len + 31) & ~31u;
  const int sum = scan_lanes((int)x.vlen, a.K);
  x.lead = a.off[0];
  x.rows_end = a.off[kMaxK];
  x.M = a.M;
  x.vlead = ((unsigned)x.lead + 31) & ~31u;
  x.vstart = x.vlead + (unsigned)sum - x.vlen;
  x.tasks_end = x.vlead + (unsigned)__builtin_amdgcn_readlane(sum, a.K - 1);
  return x;
}
template <typename Args>
__device__ __forceinline__ RowPiece find_piece(const Args& a, const RowAxis& x, unsigned v0) {
  if (__builtin_expect(a.K <= kFewTasks, 1)) {
    RowPiece p{a.M - 1, 0, -1};
    unsigned vstart = 0;
    int prev = 0;
    for (int r = 0; r < a.K + 2; ++r) {
      const int b1 = r <= a.K ? a.off[r] : a.M;
      const int len = b1 - prev;
      const unsigned o = v0 - vstart;
      if (v0 >= vstart && o < (unsigned)len) p = RowPiece{prev + (int)o, len - (int)o < 32 ? len - (int)o : 32, r >= 1 && r <= a.K ? r - 1 : -1};
      vstart += ((unsigned)len + 31) & ~31u;
      prev = b1;
    }
    return p;
  }
  int first = 0, len = x.lead, task = -1;
  unsigned o = v0;
  if (v0 >= x.tasks_end) {
    first = x.rows_end;
    len = x.M - x.rows_end;
    o = v0 - x.tasks_end;
  } else if (v0 >= x.vlead) {
    task = __builtin_ctzll(__ballot(v0 >= x.vstart && v0 - x.vstart < x.vlen));
    first = __builtin_amdgcn_readlane(x.off, task);
    len = __builtin_amdgcn_readlane(x.len, task);
    o = v0 - (unsigned)__builtin_amdgcn_readlane((int)x.vstart, task);
  }
  if (o >= (unsigned)len) return RowPiece{x.M - 1, 0, -1};
  return RowPiece{first + (int)o, len - (int)o < 32 ? len - (int)o : 32, task};
}

// The packed axis (many short tasks, see packed_rows): the rows themselves, 32 at a time, whatever their tasks
__device__ __forceinline__ RowPiece packed_piece(int M, unsigned v0) {
  const int left = M - (int)v0;
  return left > 0 ? RowPiece{(int)v0, left < 32 ? left : 32, -1} : RowPiece{M - 1, 0, -1};
}
// ... the tasks of rows [row, row + n): k from first() on, as long as their rows begin inside
struct TaskWalk {
  int off;                 // lane k: first row of task k (entries from K on: the end of the last one's rows)
};
template <typename Args>
__device__ __forceinline__ TaskWalk task_walk(const Args& a) {
  return TaskWalk{a.off[threadIdx.x & 63]};
}
__device__ __forceinline__ int task_begin(const TaskWalk& w, int k, int rows_end) {
  return k < 64 ? __builtin_amdgcn_readlane(w.off, k) : rows_end;
}
// the first task whose rows end behind `row`
template <typename Args>
__device__ __forceinline__ int first_task(const Args& a, int row) {
  const int lane = threadIdx.x & 63;
  return __builtin_popcountll(__ballot(lane < a.K && a.off[lane + 1] <= row));
}

// rows of a block of the low-rank kernels: task and row range of block b when tasks are cut into
// blocks of TM rows
template <int TM, typename Args>
__device__ __forceinline__ int rows_block(const Args& a, int b, int* lo, int* hi) {
  if (__builtin_expect(a.K <= kFewTasks, 1)) {
    int first = a.off[0];
    for (int k = 0; k < a.K; ++k) {
      const int end = a.off[k + 1], nb = (end - first + TM - 1) / TM;
      if (b < nb) {
        *lo = first + b * TM;
        *hi = end < *lo + TM ? end : *lo + TM;
        return k;
      }
      b -= nb;
      first = end;
    }
    return -1;
  }
  const int lane = threadIdx.x & 63;
  const int off = a.off[lane], len = lane < a.K ? a.off[lane + 1] - off : 0;
  const int nb = (len + TM - 1) / TM, first = scan_lanes(nb, a.K) - nb;
  const unsigned long long mine = __ballot(b >= first && b < first + nb);
  if (mine == 0) return -1;
  const int k = __builtin_ctzll(mine);
  const int o = (b - __builtin_amdgcn_readlane(first, k)) * TM, left = __builtin_amdgcn_readlane(len, k) - o;
  *lo = __builtin_amdgcn_readlane(off, k) + o;
  *hi = *lo + (left < TM ? left : TM);
  return k;
}

// task of row i (off[0] <= i < off[K]); the first lanes of a wave, or all, call this with rows in ascending order (tasks
// whose lane has left are not counted by the vote, and the walk behind it goes on from the count)
template <typename Args>
__device__ __forceinline__ int task_of_row(const Args& a, int i) {
  int k = 0;
  if (a.K > kFewTasks) {
    // where the wave's first row stands: as many tasks as end at or before it
    const int lane = threadIdx.x & 63, first = __builtin_amdgcn_readfirstlane(i);
    k = __builtin_popcountll(__ballot(lane < a.K && a.off[lane + 1] <= first));
  }
  while (i >= a.off[k + 1]) ++k;
  return k;
}

}  // namespace rowaxis
}  // namespace mlora
