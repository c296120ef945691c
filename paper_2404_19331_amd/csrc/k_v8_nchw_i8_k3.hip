#define FCM_DT TI8
#define FCM_DT_NAME "i8"
#define FCM_NCHW 1
#define FCM_K 3
#define FCM_KNAME "3"
#define FCM_TABLE_FN variants_v8_nchw_i8_k3
#define FCM_V8_TABLE FCM_V8(1, 0, 1), FCM_V8(1, 2, 1), FCM_V8(1, 4, 1), FCM_V8(3, 0, 1), FCM_V8(3, 6, 1), FCM_V8(3, 10, 1)
#include "k_v8.inc"
