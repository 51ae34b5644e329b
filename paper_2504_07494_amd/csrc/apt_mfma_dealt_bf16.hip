#define APT_MFMA_DT 2
#define APT_MFMA_DEAL true
#include "apt_mfma.inc"
