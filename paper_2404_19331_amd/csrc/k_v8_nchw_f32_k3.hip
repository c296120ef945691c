#define FCM_DT TF32
#define FCM_DT_NAME "f32"
#define FCM_NCHW 1
#define FCM_K 3
#define FCM_KNAME "3"
#define FCM_TABLE_FN variants_v8_nchw_f32_k3
#define FCM_V8_TABLE FCM_V8(2, 0, 1), FCM_V8(2, 2, 1), FCM_V8(2, 4, 1), FCM_V8(4, 0, 1), FCM_V8(4, 2, 1), FCM_V8(4, 4, 1), FCM_V8(6, 0, 1), FCM_V8(6, 2, 1), FCM_V8(6, 6, 1)
#include "k_v8.inc"
