// Test harness (CPU only): the rule that picks a direct launch's workgroups.
#include "../../paper_2609_21848_amd/csrc/internal.h"

extern "C" int direct_is_narrow(int n_items, unsigned long long wedges, unsigned long long max_work, int max_key,
                                int cus) {
  return dbbc::narrow_direct(n_items, wedges, max_work, max_key, cus) ? 1 : 0;
}
