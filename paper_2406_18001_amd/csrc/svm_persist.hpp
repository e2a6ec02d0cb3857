// One-launch K-SVM solve of small dense problems (svm_persist.hip).
#pragma once

#include "common.hpp"

namespace kdcd {

constexpr int32_t kPersistEmptyWord = 0x7ff4dead;   // both halves of an empty exchange word
constexpr int32_t kPersistGaveUp = -1000;           // status: a wait ran out, alpha must be restored
constexpr int32_t kPersistPolls = 1 << 20;          // a second and more
// Shorter solves keep their ordinary launches: an outer iteration saves 5.5 us or more, the
// start costs 20 us more.
constexpr int64_t kPersistMinOuter = 16;

struct SvmPersistArgs {
    const kdcd_matrix *A;
    const double *y, *norms;
    KParams kp;
    double nu, omega;
    int32_t s;
    int64_t H;
    const int32_t *idx;
    double *alpha, *trace;   // trace: H updates or null
    uint64_t *slots;         // 3 * groups * s words, every half kPersistEmptyWord
    int32_t *status;
    int32_t polls;           // rounds of a wait before the launch gives up
};
// Workgroups of the launch, or 0 when the problem is not one for it (also when they
// would not all be resident).
int64_t svm_persist_groups(const kdcd_matrix *A, int kind, int32_t s, int64_t n_outer);
hipError_t launch_svm_persist(const SvmPersistArgs &a, int64_t groups, hipStream_t st);

}  // namespace kdcd
