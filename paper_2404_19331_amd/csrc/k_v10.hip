// Instances of the DW->PW kernels for few pixels (fcm_kernels_v10.h): 16-pixel blocks and output-channel tiles of a
// workgroup, stride.
#include "fcm_kernels_v10.h"

namespace fcm {

#define FCM_V10S(PBK, CT, S)                                                                \
  Variant{FAM_DWPW, DT_BF16, 3, S, 16 * PBK, 0, 16 * CT, 0, 0, &launch_few10<PBK, CT>,      \
          "k_dwpw10<" #PBK "," #CT "," #S ">", 1, 16 * PBK, 10, 0, 1, PBK}
#define FCM_V10(PBK, CT) FCM_V10S(PBK, CT, 1), FCM_V10S(PBK, CT, 2)

static const Variant kTable[] = {FCM_V10(1, 1), FCM_V10(1, 2), FCM_V10(1, 4), FCM_V10(1, 8), FCM_V10(2, 2),
                                 FCM_V10(2, 4), FCM_V10(4, 2)};

const Variant* variants_v10_bf16(int* count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace fcm
