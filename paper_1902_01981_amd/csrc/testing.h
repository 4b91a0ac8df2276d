// What the tests reach beside include/codedreduce.h; not part of the interface.
#pragma once
#include "codedreduce.h"

#ifdef __cplusplus
extern "C" {
#endif

// How often a workgroup of a crew asks for what another has not published yet before it works it out itself (64 from the start, polls >= 0):
// tests take the waiting away.  CR_E_INVAL for a NULL plan or fewer than no polls.
int cr_testing_patience(cr_plan_t *plan, int polls);

#ifdef __cplusplus
}
#endif
