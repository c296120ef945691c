#define FCM_DT TF32
#define FCM_DT_NAME "f32"
#define FCM_TABLE_FN variants_v9_f32
#include "k_v9.inc"
