// Block height of causal attention: 128 query rows per workgroup, or 64, which
// doubles the workgroups and makes the longest one's chain of key tiles shorter
// per tile. No HIP in here: the rule runs on the host, and in the kernel where
// only the device knows the positions (constexpr functions compile for both).
#pragma once

namespace daf {

// Above this many 128-row blocks times heads ("jobs") the slots of the chip are
// full with 128 rows, and the doubled K/V copies per row cost more.
constexpr int narrow_most(int head_dim) { return head_dim == 128 ? 448 : 544; }
// Up to this many jobs 64 rows are never slower: their workgroups are resident at
// once (two per CU; D = 64: four) with room for the dispatcher's unevenness.
constexpr int narrow_always(int head_dim) { return head_dim == 128 ? 256 : 384; }

// Whether `jobs` blocks take 64 rows. `share`: their mean chain of key tiles over
// the longest (0.5 for a triangle, towards 1 for rows at the end of long keys).
// Beyond narrow_always 64 rows gain only where the first workgroups leave early;
// the lines follow the jobs' total work, with a step where D = 64 fills its 1024
// slots. Times with 64 rows over those with 128, rows at the end of a key
// sequence:
//   D = 128  jobs  share 0.50  0.57  0.63  0.69  0.75  0.83  0.92
//             252        0.74  0.73  0.75  0.76  0.77  0.81  0.79
//             280        0.76  0.75  0.77  0.89  1.02  1.25  1.18
//             336        0.76  0.87  0.97  1.09  1.21  1.24  1.17
//             392        0.87  0.97  1.05  1.15  1.19  1.21  1.28
//             448        0.96  1.03  1.11  1.15  1.17  1.20  1.26
//             504        1.01  1.09  1.15  1.16  1.17  1.19  1.24
//   D = 64    384        0.79  0.78  0.80  0.85  0.92  0.92  0.93
//             416        0.79  0.81  0.86  0.92  0.99  1.04  1.09
//             448        0.82  0.84  0.89  0.96  1.01  1.05  1.09
//             480        0.82  0.86  0.93  1.00  1.02  1.06  1.09
//             504        0.87  0.92  0.98  1.02  1.05
//             512        0.93  1.01  1.09  1.12  1.14  1.19  1.23
//             544        0.96  1.03  1.09  1.09  1.07  1.05  1.04
constexpr bool narrow_pays(int head_dim, long long jobs, double share) {
  if (jobs > narrow_most(head_dim)) return false;
  const double line = head_dim == 128 ? 1.06 : jobs <= 504 ? 1.27 : 1.17;
  return jobs <= narrow_always(head_dim) || share + (double)jobs / 820 <= line;
}

}  // namespace daf
